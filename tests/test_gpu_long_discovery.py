"""GPU: first calls with so many rounds that they go on by captured chunks (from
2,048 rounds on): the last direct chunk, the first and second captured ones, a chunk
size that does not divide, and a call in another mode on the same handle between two
that search for the round count.  Exact equality with the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("algorithm", ["push", "pull"])
@pytest.mark.parametrize("chunk", [16, 100])
@pytest.mark.parametrize("n", [4_060, 4_098, 4_140, 4_600])  # n // 2 + 1 rounds
def test_first_calls_with_many_rounds(n, chunk, algorithm):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] long discovery {n} chunk={chunk} {algorithm}", flush=True)
    g = graphgen.path(n)
    ref = oracle.rsc(g.rowptr, g.colidx)
    sizes = np.cumsum(np.bincount(ref.round_of, minlength=ref.rounds + 1)[::-1])[::-1][1:]
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    with gc.Graph(rp, ci, algorithm=algorithm, chunk_rounds=chunk, wait_polls=0) as G:
        for i in range(3):
            out = G.color()
            if i == 0:  # (the round count stays unknown: nobody asks)
                torch.cuda.synchronize()
            else:
                assert G.stats() == (ref.rounds, 2)
                assert np.array_equal(G.round_sizes(), sizes)
            assert np.array_equal(out.cpu().numpy(), ref.colors)
            if i == 0:
                G.set("lanes", 4)  # (the captured chunk no longer fits)
