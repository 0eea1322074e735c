"""GPU: one-launch passes whose waits give up (GC_OPT_WAIT_POLLS = 1, so that the
first wait for another workgroup does) still colour the graph: calls that find
the round count and calls that know it, with and without a look at the result
between them; the handle then goes on without the pass until the option is set
again.  Also the passes turned off.  Exact equality with the oracle's colours,
rounds and round sizes."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {
    "resident": lambda: graphgen.er(10_000, 100_000, 5),
    "resident_24576": lambda: graphgen.er(24_576, 150_000, 6),
    "resident_many_rounds": lambda: graphgen.er(600, 26_000, 8),
    "core_4096": lambda: graphgen.er(4096, 350_000, 4),
    "core_K512": lambda: graphgen.complete(512),
    "core_late": lambda: graphgen.rmat(15, 16, seed=3),
    "core_wide_state": lambda: graphgen.star(40_000, 20_000),
    "core_late_dense": lambda: graphgen.er(5000, 1_500_000, 6),
}
WAITED = {"core_wide_state"}  # two rounds: no late core once the rounds are known


def _check(G, out, ref, sizes, what):
    assert G.stats() == (ref.rounds, int(ref.colors.max()) + 1), what
    assert np.array_equal(out.cpu().numpy(), ref.colors), what
    assert np.array_equal(G.round_sizes(), sizes), what


@pytest.mark.parametrize("rp64", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_pass_that_gives_up(name, rp64):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] gives up {name} rp64={rp64}", flush=True)
    g = CASES[name]()
    ref = oracle.rsc(g.rowptr, g.colidx)
    sizes = np.cumsum(np.bincount(ref.round_of, minlength=ref.rounds + 1)[::-1])[::-1][1:]
    rp = torch.from_numpy(g.rowptr.astype(np.int64 if rp64 else np.int32)).cuda()
    ci = torch.from_numpy(g.colidx).cuda()
    with gc.Graph(rp, ci, wait_polls=1) as G:  # R unknown
        _check(G, G.color(), ref, sizes, "first")
        assert name in WAITED or G.get(gc.GC_OPT_WAIT_POLLS) == 0
    with gc.Graph(rp, ci) as G:
        for what in ("first", "second"):
            _check(G, G.color(), ref, sizes, what)
        assert G.get(gc.GC_OPT_WAIT_POLLS) == 1 << 20
        for turn in range(2):
            G.set("wait_polls", 1)
            outs = [G.color() for _ in range(3)]  # R known, nobody looks in between
            torch.cuda.synchronize()
            for out in outs:
                assert np.array_equal(out.cpu().numpy(), ref.colors), turn
            _check(G, outs[-1], ref, sizes, turn)
            assert name in WAITED or G.get(gc.GC_OPT_WAIT_POLLS) == 0
            _check(G, G.color(), ref, sizes, "by the rounds")
        G.set("wait_polls", 0)
        _check(G, G.color(), ref, sizes, "off")
        G.set("wait_polls", 1 << 20)
        for what in ("again", "and again"):
            _check(G, G.color(), ref, sizes, what)
        assert G.get(gc.GC_OPT_WAIT_POLLS) == 1 << 20


def test_wait_polls_range():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    g = graphgen.path(10)
    with gc.Graph(torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()) as G:
        for bad in (-1, 1 << 31):
            with pytest.raises(gc.GCError):
                G.set("wait_polls", bad)
