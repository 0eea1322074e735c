"""GPU: a handle that learned its round count under another driver, profiling or a
turned-off core pass still takes the core pass for the last rounds of its default
calls (seen from a wait that gives up at once), with the same result."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("first", ["graph", "host", "chunked", "persistent", "profile", "off"])
def test_core_round_learned_under(first):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] core round learned under {first}", flush=True)
    g = graphgen.rmat(15, 16, seed=3)
    ref = oracle.rsc(g.rowptr, g.colidx)
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    with gc.Graph(rp, ci) as G:
        name, value, back = {"profile": ("profile", 1, 0), "off": ("wait_polls", 0, 1 << 20)}.get(
            first, ("mode", first, "graph"))
        G.set(name, value)
        G.color()
        assert G.stats()[0] == ref.rounds
        G.set(name, back)
        for polls in (1 << 20, 1):
            G.set("wait_polls", polls)
            out = G.color()
            assert G.stats() == (ref.rounds, int(ref.colors.max()) + 1)
            assert np.array_equal(out.cpu().numpy(), ref.colors)
        assert G.get(gc.GC_OPT_WAIT_POLLS) == 0
