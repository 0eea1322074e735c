"""GPU: first calls with so many rounds that they go on by graphs of chunks (from
2,048 rounds on): the last direct chunk, the first and second graphs, a chunk
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
                G.set("lanes", 4)  # (the graph no longer fits)


@pytest.mark.parametrize("n", [32_766, 32_768, 32_770, 65_600])  # n // 2 + 1 rounds
def test_known_rounds_beyond_one_chunk(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] many known rounds {n}", flush=True)
    g = graphgen.path(n)
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    want = torch.arange(n, dtype=torch.int32, device="cuda") % 2
    sizes = n - 2 * np.arange(n // 2 + 1)  # in each round the two lowest ids left (one in the first)
    sizes[1:] += 1
    with gc.Graph(rp, ci, wait_polls=0) as G:
        for _ in range(3):
            out = G.color()
            assert G.stats() == (n // 2 + 1, 2)
            assert torch.equal(out, want)
            assert np.array_equal(G.round_sizes(), sizes)
