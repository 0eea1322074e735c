"""GPU: the resident pass (a whole colouring in one launch, the graph's rows and
states in LDS) at the edges of its ranges: chunk and workgroup remainders, the
largest graph (24,576 vertices) and one vertex more, colours on both sides of
bit 64 of a vertex's mask, the largest degree with one-byte states, many rounds,
rows that fit on average but not in one workgroup (the rounds' own passes take
over), a graph changed in place, and four calls side by side.  Exact equality
with the oracle's colours, rounds and round sizes."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _uneven():
    # the rows of one workgroup's chunks (0, 64, 128, ...) hold most entries
    n, rng = 20_032, np.random.default_rng(4)
    edges = set()
    for c in range(0, n // 64, 64):
        for v in range(64 * c, 64 * c + 64):
            for u in rng.integers(0, n, 110):
                if u // 64 % 64:
                    edges.add((min(v, int(u)), max(v, int(u))))
    return graphgen.from_edges(n, edges)


CASES = {
    "one": lambda: graphgen.empty(1),
    "edgeless": lambda: graphgen.empty(130),
    "n63": lambda: graphgen.er(63, 400, 1),
    "n64": lambda: graphgen.er(64, 400, 2),
    "n65": lambda: graphgen.er(65, 400, 3),
    "n4095": lambda: graphgen.er(4095, 60_000, 4),
    "n4097": lambda: graphgen.er(4097, 60_000, 5),
    "n24576": lambda: graphgen.er(24_576, 150_000, 6),
    "n24577": lambda: graphgen.er(24_577, 150_000, 7),
    "dense": lambda: graphgen.er(600, 26_000, 8),     # degrees up to about 110
    "K100": lambda: graphgen.complete(100),
    "K127": lambda: graphgen.complete(127),
    "path": lambda: graphgen.path(3000),
    "uneven": _uneven,
}


def _bind(gc, g, rows_sorted, rp64):
    h = g if rows_sorted else graphgen.shuffle_rows(g, np.random.default_rng(1))
    rp = torch.from_numpy(h.rowptr.astype(np.int64 if rp64 else np.int32)).cuda()
    ci = torch.from_numpy(h.colidx if h.nnz else np.zeros(0, np.int32)).cuda()
    return rp, ci


@pytest.mark.parametrize("rp64", [False, True])
@pytest.mark.parametrize("rows_sorted", [True, False])
@pytest.mark.parametrize("name", sorted(CASES))
def test_resident_matches_oracle(name, rows_sorted, rp64):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    g = CASES[name]()
    ref = oracle.rsc(g.rowptr, g.colidx)
    sizes = np.cumsum(np.bincount(ref.round_of, minlength=ref.rounds + 1)[::-1])[::-1][1:]
    print(f"[case] resident {name} sorted={rows_sorted} rp64={rp64}", flush=True)
    rp, ci = _bind(gc, g, rows_sorted, rp64)
    with gc.Graph(rp, ci, rows_sorted=rows_sorted) as G:
        for mode in ("graph", "graph", "host", "graph"):
            G.set("mode", mode)
            out = G.color()
            assert G.stats() == (ref.rounds, int(ref.colors.max()) + 1)
            assert np.array_equal(out.cpu().numpy(), ref.colors)
            assert np.array_equal(G.round_sizes(), sizes)


def test_resident_reports_a_changed_graph():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    many = graphgen.path(5000)
    rp, ci = _bind(gc, many, True, False)
    keep_rp, keep_ci = rp.clone(), ci.clone()
    rp.zero_()  # edgeless: one round
    with gc.Graph(rp, ci) as G:
        G.color()
        assert G.stats()[0] == 1
        rp.copy_(keep_rp)
        ci.copy_(keep_ci)
        G.color()
        with pytest.raises(gc.GCError) as e:
            G.stats()
        assert e.value.code == gc.GC_EINVAL


def test_four_residents_side_by_side():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    g = graphgen.er(24_000, 180_000, 9)
    ref = oracle.rsc(g.rowptr, g.colidx)
    rp, ci = _bind(gc, g, True, False)
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
