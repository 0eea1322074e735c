"""GPU: batch launches inside a captured graph, whose set-up calls (the kernels'
LDS size) are made on every launch: a batch and a resumable step, replayed several
times with eager calls and a wait between the replays, each against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_batch_and_step_replayed():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    gs = [graphgen.er(n, 6 * n, n) for n in (40, 900, 5000, 60_000)] + [graphgen.rmat(11, 16, seed=2)]
    refs = [oracle.rsc(g.rowptr, g.colidx) for g in gs]
    want = torch.from_numpy(np.concatenate([r.colors for r in refs])).cuda()
    rounds_want = [r.rounds for r in refs]
    voff = np.cumsum([0] + [g.n for g in gs]).astype(np.int64)
    eoff = np.cumsum([0] + [g.nnz for g in gs]).astype(np.int64)
    rp = torch.from_numpy(np.concatenate([g.rowptr for g in gs]).astype(np.int32)).cuda()
    ci = torch.from_numpy(np.concatenate([g.colidx for g in gs])).cuda()
    args = (torch.from_numpy(voff).cuda(), torch.from_numpy(eoff).cuda(), rp, ci)
    rows = [(int(voff[i] + i), int(eoff[i]), int(voff[i]), gs[i].n, 0) for i in range(len(gs))]
    fresh = torch.from_numpy(gc.desc_array(rows).view(np.uint8)).cuda()
    descs = fresh.clone()
    stepped = torch.empty_like(want)
    ws = torch.empty(gc.gc_batch_step_workspace_bytes(len(gs), 0), dtype=torch.uint8, device="cuda")

    def run():
        colors, rounds = gc.color_batch(*args, voff_host=voff, eoff_host=eoff)
        descs.copy_(fresh)
        gc.batch_step(descs, rp, ci, stepped, 0, workspace=ws)
        return colors, rounds

    def check(colors, rounds, what):
        assert torch.equal(colors, want), what
        assert torch.equal(stepped, want), what
        assert rounds.cpu().tolist() == rounds_want, what

    check(*run(), "eager")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        colors, rounds = run()
    for i in range(4):
        colors.fill_(7)
        stepped.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        check(colors, rounds, i)
        other = gc.color_batch(*args, voff_host=voff, eoff_host=eoff)
        assert torch.equal(other[0], want)
