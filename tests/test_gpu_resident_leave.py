"""GPU: workgroups of the resident pass that leave one after the other.  The
chunk of 64 vertices that a workgroup owns holds a clique of its own size, so in
every round one of them colours its last vertex and leaves while the others go
on, down to a single one.  Many calls in a row and four side by side; exact
equality with the oracle's colours, rounds and round sizes."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _staggered(per_workgroup):
    # workgroup g owns chunks g, g + 64, ...: cliques of g + 1 vertices in each
    edges = [(64 * c + i, 64 * c + j) for c in range(64 * per_workgroup)
             for i in range(c % 64 + 1) for j in range(i)]
    return graphgen.from_edges(64 * 64 * per_workgroup, edges)


@pytest.mark.parametrize("per_workgroup", [1, 6])
def test_workgroups_leave_one_by_one(per_workgroup):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] staggered {per_workgroup}", flush=True)
    g = _staggered(per_workgroup)
    ref = oracle.rsc(g.rowptr, g.colidx)
    sizes = np.cumsum(np.bincount(ref.round_of, minlength=ref.rounds + 1)[::-1])[::-1][1:]
    assert ref.rounds == 64
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    want = torch.from_numpy(ref.colors).cuda()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(4)]
    graphs = [gc.Graph(rp, ci) for _ in streams]
    for _ in range(20):  # alone
        out = graphs[0].color()
        assert graphs[0].stats() == (ref.rounds, int(ref.colors.max()) + 1)
        assert torch.equal(out, want)
        assert np.array_equal(graphs[0].round_sizes(), sizes)
    for G in graphs:
        G.color()
        G.stats()
    outs = []
    for _ in range(20):  # side by side
        for G, s in zip(graphs, streams):
            with torch.cuda.stream(s):
                outs.append(G.color())
    torch.cuda.synchronize()
    assert all(torch.equal(o, want) for o in outs)
    for G in graphs:
        assert G.stats()[0] == ref.rounds
        assert np.array_equal(G.round_sizes(), sizes)
        G.close()
