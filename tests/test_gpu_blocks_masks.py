"""GPU: the p-block passes with masks in the place of the slots, at the edges of
their ranges: block sizes around each word of a unit (63 .. 65, 127 .. 129,
255 .. 257 vertices; 257 takes the slots), blocks of one vertex, more blocks
than vertices, colours on both sides of bit 64 of the mask, the largest degree
with one-byte states (126) and the first beyond it, and a round cap.  Exact
equality with the oracle's colours, rounds and round sizes."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRAPHS = {
    "er": lambda: graphgen.er(2570, 30_000, 1),
    "er_dense": lambda: graphgen.er(300, 12_000, 2),      # degrees around 80: colours beyond 32
    "K100": lambda: graphgen.complete(100),               # colours 0..99
    "K127": lambda: graphgen.complete(127),               # maximum degree 126
    "K128": lambda: graphgen.complete(128),               # two-byte states: the passes with slots
    "path": lambda: graphgen.path(1000),                  # every neighbour in the own block
}


@pytest.mark.parametrize("per_block", [1, 2, 31, 63, 64, 65, 127, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_masks_match_oracle(name, per_block):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    g = GRAPHS[name]()
    for p in {max(1, -(-g.n // per_block)), g.n + 3 if per_block == 1 else 1}:
        print(f"[case] blocks masks {name} p={p}", flush=True)
        want, R, rec = oracle.blocks(g.rowptr, g.colidx, p)
        sizes = [int((rec >= r - 1).sum()) for r in range(1, R + 1)]
        h = graphgen.shuffle_rows(g, np.random.default_rng(2))
        rp, ci = torch.from_numpy(h.rowptr).cuda(), torch.from_numpy(h.colidx).cuda()
        with gc.Graph(rp, ci, rows_sorted=False, algorithm="blocks", partitions=p) as G:
            for _ in range(2):
                out = G.color()
                assert G.stats() == (R, int(want.max()) + 1)
                assert np.array_equal(out.cpu().numpy(), want)
            assert list(G.round_sizes()) == sizes
            if R > 2:
                G.set("max_rounds", 2)
                G.color()
                with pytest.raises(gc.GCError) as e:
                    G.stats()
                assert e.value.code == gc.GC_EROUNDS
