"""GPU: gc_get_stats of a call read after the algorithm was switched: the next call
must not take the other colouring's round count for its own."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n, m", [(10_000, 100_000), (60_000, 600_000)])
def test_stats_read_after_a_switch(n, m):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    g = graphgen.er(n, m, 5)
    ref = oracle.rsc(g.rowptr, g.colidx)
    seq = oracle.seq(g.rowptr, g.colidx)
    want = {"auto": (ref.rounds, ref.colors), "seq": (oracle.seq_rounds(g.rowptr, g.colidx)[0], seq)}
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    with gc.Graph(rp, ci) as G:
        for now, then in (("auto", "seq"), ("seq", "auto"), ("auto", "auto")):
            print(f"[case] stats after a switch {now} -> {then}", flush=True)
            out = G.color()
            G.set("algorithm", then)
            assert G.stats()[0] == want[now][0]
            assert np.array_equal(out.cpu().numpy(), want[now][1])
