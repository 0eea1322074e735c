"""GPU: the data-flow pass of GC_ALGO_SEQ at the sizes where it can go wrong:
units of one, 64 and 65 vertices, vertices of either side of the lane /
wavefront split next to each other, colour windows that slide (64 colours per
lane, 1,024 per wavefront), 32- and 64-bit words, and rounds beyond the ones
counted in LDS (2,048) and beyond the trace (65,536).  Exact equality with the
oracle's colours, rounds and round sizes."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _hubs():
    # wavefront-class vertices scattered among light ones, two of them adjacent ids
    rng = np.random.default_rng(5)
    edges = {(min(a, b), max(a, b)) for a, b in rng.integers(0, 700, (2500, 2)) if a != b}
    for hub in (0, 63, 64, 65, 300, 301, 699):
        edges |= {(min(hub, int(u)), max(hub, int(u))) for u in rng.integers(0, 700, 200) if u != hub}
    return graphgen.from_edges(700, edges)


def _wide_star():
    # colours and rounds need 17 + 17 bits: 64-bit words
    return graphgen.star(70_000, 35_000)


CASES = {
    "one": (lambda: graphgen.empty(1), {}),
    "path64": (lambda: graphgen.path(64), {}),
    "path65": (lambda: graphgen.path(65), {}),
    "hubs": (_hubs, {}),
    "hubs_all_wavefront": (_hubs, {"medium_degree": 1}),
    "window_lane": (lambda: graphgen.complete(200), {"medium_degree": 1000}),
    "window_wave": (lambda: graphgen.complete(1100), {}),
    "rounds_past_lds": (lambda: graphgen.path(2500), {}),
    "rounds_past_trace": (lambda: graphgen.path(66_001), {}),
    "words64": (_wide_star, {}),
}


@pytest.mark.parametrize("rp64", [False, True])
@pytest.mark.parametrize("rows_sorted", [True, False])
@pytest.mark.parametrize("name", sorted(CASES))
def test_flow_matches_oracle(name, rows_sorted, rp64):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    make, options = CASES[name]
    g = make()
    h = g if rows_sorted else graphgen.shuffle_rows(g, np.random.default_rng(1))
    print(f"[case] seq flow {name} sorted={rows_sorted} rp64={rp64}", flush=True)
    want = oracle.seq(g.rowptr, g.colidx)
    R, when = oracle.seq_rounds(g.rowptr, g.colidx)
    sizes = np.cumsum(np.bincount(when, minlength=R + 1)[::-1])[::-1][1:]
    rp = torch.from_numpy(h.rowptr.astype(np.int64 if rp64 else np.int32)).cuda()
    ci = torch.from_numpy(h.colidx).cuda()
    with gc.Graph(rp, ci, rows_sorted=rows_sorted, algorithm="seq", **options) as G:
        for _ in range(2):
            out = G.color()
            assert G.stats() == (R, int(want.max()) + 1)
            assert np.array_equal(out.cpu().numpy(), want)
        assert np.array_equal(G.round_sizes(), sizes[:gc.GC_TRACE_ROUNDS])
