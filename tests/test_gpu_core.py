"""GPU: the core pass (the last rounds, or all rounds of a small graph with
degrees above 126, in one launch) at the edges of its ranges: workgroup
remainders (191, 192, 193 vertices),
the largest core (4,096 vertices) and one vertex more, the last colour with a
mask bit (511) and the first without, rows long enough for a whole workgroup,
all three state widths, both row layouts and offset widths, pushed and
gathered rounds before it, and calls that know the round count.  Exact equality
with the oracle's colours, rounds and round sizes."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _clique_over_leaves(k, leaves):
    # k pairwise adjacent vertices above `leaves` vertices that all of them touch
    edges = [(u, leaves + i) for i in range(k) for u in range(leaves)]
    edges += [(leaves + i, leaves + j) for i in range(k) for j in range(i)]
    return graphgen.from_edges(leaves + k, edges)


CASES = {
    "n191": lambda: graphgen.er(191, 16_500, 1),
    "n192": lambda: graphgen.er(192, 16_500, 2),
    "n193": lambda: graphgen.er(193, 16_500, 3),
    "star": lambda: graphgen.star(200, 100),
    "n4096": lambda: graphgen.er(4096, 350_000, 4),
    "n4097": lambda: graphgen.er(4097, 350_000, 5),
    "dense": lambda: graphgen.er(5000, 1_500_000, 6),
    "K512": lambda: graphgen.complete(512),
    "K513": lambda: graphgen.complete(513),
    "star_wide_state": lambda: graphgen.star(40_000, 20_000),
    "long_rows": lambda: _clique_over_leaves(20, 8_500),
    "rmat": lambda: graphgen.rmat(15, 16, seed=3),
}


@pytest.mark.parametrize("algorithm", ["push", "pull"])
@pytest.mark.parametrize("rows_sorted", [True, False])
@pytest.mark.parametrize("name", sorted(CASES))
def test_core_matches_oracle(name, rows_sorted, algorithm):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    g = CASES[name]()
    ref = oracle.rsc(g.rowptr, g.colidx)
    sizes = np.cumsum(np.bincount(ref.round_of, minlength=ref.rounds + 1)[::-1])[::-1][1:]
    h = g if rows_sorted else graphgen.shuffle_rows(g, np.random.default_rng(1))
    for rp64 in (False, True):
        print(f"[case] core {name} sorted={rows_sorted} {algorithm} rp64={rp64}", flush=True)
        rp = torch.from_numpy(h.rowptr.astype(np.int64 if rp64 else np.int32)).cuda()
        ci = torch.from_numpy(h.colidx).cuda()
        with gc.Graph(rp, ci, rows_sorted=rows_sorted, algorithm=algorithm) as G:
            for mode in ("graph", "graph", "graph", "host", "graph"):
                G.set("mode", mode)
                out = G.color()
                assert G.stats() == (ref.rounds, int(ref.colors.max()) + 1)
                assert np.array_equal(out.cpu().numpy(), ref.colors)
                assert np.array_equal(G.round_sizes(), sizes)


def test_core_on_four_streams_at_once():
    """Four handles whose cores run side by side, several calls each."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    g = graphgen.er(4096, 350_000, 7)
    ref = oracle.rsc(g.rowptr, g.colidx)
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(4)]
    graphs = [gc.Graph(rp, ci) for _ in streams]
    for G in graphs:
        G.color()
        G.stats()
    outs = []
    for _ in range(5):
        for G, s in zip(graphs, streams):
            with torch.cuda.stream(s):
                outs.append(G.color())
    torch.cuda.synchronize()
    assert all(np.array_equal(o.cpu().numpy(), ref.colors) for o in outs)
    for G in graphs:
        assert G.stats()[0] == ref.rounds
        G.close()
