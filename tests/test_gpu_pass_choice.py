"""GPU: the choice between a one-launch pass and the rounds' own passes on both sides
of its lines: graphs without edges, few rounds on a small graph, nearly complete
graphs, and many light rounds on a graph that the resident pass could take.  Exact
equality with the oracle's colours, rounds and round sizes on every call; whether
the core or resident pass ran is seen from a wait that gives up at once."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _cliques(k, q):
    j = np.arange(k)
    rows = np.stack([np.delete(j, i) for i in range(k)]).reshape(1, -1) + k * np.arange(q)[:, None]
    return graphgen.CSR(np.arange(k * q + 1, dtype=np.int64) * (k - 1),
                        rows.reshape(-1).astype(np.int32))


def _paths(length, q):
    p = graphgen.path(length)
    ci = (p.colidx[None] + length * np.arange(q)[:, None]).reshape(-1).astype(np.int32)
    rp = np.concatenate([p.rowptr[:-1][None] + p.nnz * np.arange(q)[:, None]], axis=1).reshape(-1)
    return graphgen.CSR(np.append(rp, p.nnz * q), ci)


# name: graph, rows sorted, whether a call with R known takes one of the passes
CASES = {
    "one vertex": (lambda: graphgen.empty(1), True, False),
    "no edges": (lambda: graphgen.empty(20_000), True, False),
    "star": (lambda: graphgen.star(3_000, 1_000), True, False),
    "9 rounds": (lambda: _cliques(9, 3), True, True),          # resident
    "K140": (lambda: graphgen.complete(140), True, True),
    "K600": (lambda: graphgen.complete(600), True, False),
    "K520 minus": (lambda: _cliques(260, 4), True, True),
    "sparse 20,480": (lambda: _cliques(5, 4_096), True, True),    # R = 5
    "paths 20,480": (lambda: _paths(40, 512), True, True),
    "paths 20,520": (lambda: _paths(40, 513), True, False),
    "cliques 16,384": (lambda: _cliques(32, 512), True, True),
    "cliques 16,416": (lambda: _cliques(32, 513), True, False),
    "cliques unsorted": (lambda: _cliques(32, 513), False, True),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_pass_choice(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] pass choice {name}", flush=True)
    make, rows_sorted, one_launch = CASES[name]
    g = make()
    ref = oracle.rsc(g.rowptr, g.colidx)
    sizes = np.cumsum(np.bincount(ref.round_of, minlength=ref.rounds + 1)[::-1])[::-1][1:]
    h = g if rows_sorted else graphgen.shuffle_rows(g, np.random.default_rng(1))
    rp = torch.from_numpy(h.rowptr).cuda()
    ci = torch.from_numpy(h.colidx if h.nnz else np.zeros(0, np.int32)).cuda()
    with gc.Graph(rp, ci, rows_sorted=rows_sorted) as G:
        for polls in (1 << 20, 1 << 20, 1, 1 << 20):
            G.set("wait_polls", polls)
            out = G.color()
            assert G.stats() == (ref.rounds, int(ref.colors.max()) + 1)
            assert np.array_equal(out.cpu().numpy(), ref.colors)
            assert np.array_equal(G.round_sizes(), sizes[:gc.GC_TRACE_ROUNDS])
            if polls == 1:
                # (a single workgroup waits for nobody, and in few rounds nobody may have to)
                gave_up = G.get(gc.GC_OPT_WAIT_POLLS) == 0
                assert one_launch or not gave_up
                assert gave_up or not one_launch or g.n <= 64 or ref.rounds < 20
    with gc.Graph(rp, ci, rows_sorted=rows_sorted, algorithm="seq") as G:
        want = oracle.seq(g.rowptr, g.colidx)
        for _ in range(2):
            out = G.color()
            assert G.stats() == (oracle.seq_rounds(g.rowptr, g.colidx)[0], int(want.max()) + 1)
            assert np.array_equal(out.cpu().numpy(), want)
