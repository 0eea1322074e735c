"""GPU: gc_get_stats of a finished call makes no device call of its own, so that
it may stand inside another stream's capture (which such a call would break), and
the handle still learns the round count from it: a graph whose last rounds a core
pass takes over, one that runs in it alone, a small one and sequential First Fit."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {
    "core_late": (lambda: graphgen.rmat(15, 16, seed=3), {}),
    "core_4096": (lambda: graphgen.er(4096, 350_000, 4), {}),
    "resident": (lambda: graphgen.er(10_000, 100_000, 5), {}),
    "rounds": (lambda: graphgen.er(60_000, 100_000, 5), {}),
    "seq": (lambda: graphgen.er(10_000, 100_000, 5), {"algorithm": "seq"}),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_stats_of_a_finished_call_inside_a_capture(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] stats in capture {name}", flush=True)
    make, options = CASES[name]
    g = make()
    if options:
        colors = oracle.seq(g.rowptr, g.colidx)
        rounds = oracle.seq_rounds(g.rowptr, g.colidx)[0]
    else:
        ref = oracle.rsc(g.rowptr, g.colidx)
        colors, rounds = ref.colors, ref.rounds
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    x = torch.zeros(64, dtype=torch.int32, device="cuda")
    with gc.Graph(rp, ci, **options) as G:
        out = G.color()
        torch.cuda.synchronize()
        G.set("profile", 0)  # the call is known to be over
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):  # (global capture mode)
            x.add_(1)
            assert G.stats() == (rounds, int(colors.max()) + 1)
        for i in range(3):
            graph.replay()
            torch.cuda.synchronize()
            assert int(x[0]) == i + 1
        assert np.array_equal(out.cpu().numpy(), colors)
        for _ in range(3):
            out = G.color()
            assert G.stats()[0] == rounds
            assert np.array_equal(out.cpu().numpy(), colors)
