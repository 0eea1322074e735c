"""GPU: the round sizes of the data-flow pass over many calls.  Every workgroup of
its finishing pass adds counts into the trace, and the last one to arrive turns
them into round sizes, so all adds have to be complete by then: rounds counted in
LDS (up to 2,048), rounds added one by one beyond them, and many workgroups."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {
    "path_6000": lambda: graphgen.path(6000),
    "er_300k": lambda: graphgen.er(300_000, 1_500_000, 3),
    "rmat": lambda: graphgen.rmat(15, 16, seed=3),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_round_sizes_over_many_calls(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] seq sizes {name}", flush=True)
    g = CASES[name]()
    R, when = oracle.seq_rounds(g.rowptr, g.colidx)
    sizes = np.cumsum(np.bincount(when, minlength=R + 1)[::-1])[::-1][1:]
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    with gc.Graph(rp, ci, algorithm="seq") as G:
        for i in range(50):
            G.color()
            assert G.stats()[0] == R
            assert np.array_equal(G.round_sizes(), sizes), i
