"""GPU: sequential First Fit where a lane walks rows of more than 64 entries: colours
on both sides of its first window (64 colours) and of the one in LDS behind it (256
more, and again after a second walk), beside small graphs in the same unit, and the
wider grid of graphs whose vertices take a wavefront each.  Exact equality with the
oracle's colours, rounds and round sizes."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _cliques(sizes):
    rows, rp, at = [], [0], 0
    for k in sizes:
        j = np.arange(at, at + k)
        rows += [np.delete(j, i) for i in range(k)]
        rp += [k - 1] * k
        at += k
    return graphgen.CSR(np.cumsum(rp).astype(np.int64), np.concatenate(rows).astype(np.int32))


CASES = {
    "windows": (lambda: _cliques([63, 64, 65, 66, 3, 319, 320, 321, 322, 5, 640, 641, 1]),
                {"medium_degree": 2000}),
    "K200": (lambda: _cliques([200] * 7), {}),
    "er_d100": (lambda: graphgen.er(3000, 150_000, 1), {}),
    "wide wavefronts": (lambda: _cliques([300] * 40), {}),
    "narrow wavefronts": (lambda: _cliques([300] * 31), {}),
}


@pytest.mark.parametrize("rp64", [False, True])
@pytest.mark.parametrize("rows_sorted", [True, False])
@pytest.mark.parametrize("name", sorted(CASES))
def test_long_light_rows(name, rows_sorted, rp64):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] seq deep {name} sorted={rows_sorted} rp64={rp64}", flush=True)
    make, options = CASES[name]
    g = make()
    want = oracle.seq(g.rowptr, g.colidx)
    R, when = oracle.seq_rounds(g.rowptr, g.colidx)
    sizes = np.cumsum(np.bincount(when, minlength=R + 1)[::-1])[::-1][1:]
    h = g if rows_sorted else graphgen.shuffle_rows(g, np.random.default_rng(1))
    rp = torch.from_numpy(h.rowptr.astype(np.int64 if rp64 else np.int32)).cuda()
    ci = torch.from_numpy(h.colidx).cuda()
    with gc.Graph(rp, ci, rows_sorted=rows_sorted, algorithm="seq", **options) as G:
        for _ in range(2):
            out = G.color()
            assert G.stats() == (R, int(want.max()) + 1)
            assert np.array_equal(out.cpu().numpy(), want)
            assert np.array_equal(G.round_sizes(), sizes)
