"""GPU: the batch kernel's pushed-colour path at the edges of its ranges: state
layouts (24 colours in a word per vertex up to 40,704 vertices, 16 colours and
3 bytes up to 54,270), vertices whose tracked colours are all taken, chunk and
packing remainders (63, 64, 65 vertices), the maximum degree at which it ends
(127 / 128), unaligned rows, and steps that resume it.  Exact equality with the
oracle's colours and rounds."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

WORD_N = 159 * 1024 // 4          # largest graph of the word layout
BYTES3_N = (159 * 1024 - 4) // 3  # largest of the 3-byte layout

CASES = {
    "chunks": lambda: [graphgen.er(n, 4 * n, n) for n in (63, 64, 65, 127, 1023, 1024, 1025)],
    "word_layout_end": lambda: [graphgen.er(WORD_N, 3 * WORD_N, 1), graphgen.er(WORD_N + 1, 3 * WORD_N, 2)],
    "bytes3_layout_end": lambda: [graphgen.er(BYTES3_N, 200_000, 3), graphgen.er(BYTES3_N + 1, 200_000, 4)],
    # 26 colours and more: beyond the masks of both layouts
    "colours_beyond_mask": lambda: [graphgen.er(1_000, 40_000, 5), graphgen.er(45_000, 1_100_000, 6)],
    "degree_edge": lambda: [graphgen.complete(128), graphgen.complete(129), graphgen.star(127, 60), graphgen.star(128, 60)],
    "long_path": lambda: [graphgen.path(777)],
}


def _pack(graphs):
    voff = np.cumsum([0] + [g.n for g in graphs]).astype(np.int64)
    eoff = np.cumsum([0] + [g.nnz for g in graphs]).astype(np.int64)
    rp = np.concatenate([g.rowptr.astype(np.int32) for g in graphs])
    ci = np.concatenate([g.colidx.astype(np.int32) for g in graphs])
    return voff, eoff, rp, ci


@pytest.mark.parametrize("step_rounds", [0, 3])
@pytest.mark.parametrize("name", sorted(CASES))
def test_pushed_batch_matches_oracle(name, step_rounds):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    graphs = CASES[name]()
    print(f"[case] batch push {name} step={step_rounds}", flush=True)
    voff, eoff, rp, ci = _pack(graphs)
    # one entry in front: rows that start at no 16-byte boundary
    d_ci = torch.from_numpy(np.concatenate([[0], ci]).astype(np.int32)).cuda()[1:]
    d_rp = torch.from_numpy(rp).cuda()
    if step_rounds == 0:
        colors, rounds = gc.color_batch(torch.from_numpy(voff).cuda(), torch.from_numpy(eoff).cuda(),
                                        d_rp, d_ci, voff_host=voff, eoff_host=eoff)
        rounds = rounds.cpu().numpy()
    else:
        colors = torch.full((int(voff[-1]),), 77, dtype=torch.int32, device="cuda")
        rows = [(int(voff[i] + i), int(eoff[i]), int(voff[i]), g.n) for i, g in enumerate(graphs)]
        descs = torch.from_numpy(gc.desc_array(rows).view(np.uint8)).cuda()
        for _ in range(1 + max(g.n for g in graphs)):
            gc.batch_step(descs, d_rp, d_ci, colors, step_rounds)
            table = descs.cpu().numpy().view(gc.DESC_DTYPE)
            if not table["active"].any():
                break
        rounds = table["rounds"]
    got = colors.cpu().numpy()
    for i, g in enumerate(graphs):
        ref = oracle.rsc(g.rowptr, g.colidx)
        assert rounds[i] == ref.rounds, (i, g.n)
        assert np.array_equal(got[voff[i]:voff[i + 1]], ref.colors), (i, g.n)
