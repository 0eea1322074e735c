"""GPU: batched colouring at the edges of the layouts that a graph's state and colour
masks take in LDS (by vertices and maximum degree), with more colours than a mask
holds, of the gathering passes beyond them, and of the kernel for many small
graphs (the largest of them, one vertex or entry more, a large graph beside them).
Whole colourings and resumed steps, against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _with_clique(n, k, seed):
    # a sparse random graph (little work: no team) with a clique of k among its vertices
    base = graphgen.er(n, int(0.4 * n), seed)
    rows = np.repeat(np.arange(n), np.diff(base.rowptr))
    ids = np.random.default_rng(seed).choice(n, k, replace=False)
    a, b = np.meshgrid(ids, ids)
    keep = a != b
    key = np.unique(np.concatenate([rows * n + base.colidx, a[keep] * n + b[keep]]))
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=rp[1:])
    return graphgen.CSR(rp, (key % n).astype(np.int32))


SLOTS = {f"{n}_K{k}": (lambda n=n, k=k: _with_clique(n, k, n + k))
         for n, k in [(40_704, 60), (40_705, 60), (54_272, 60), (54_273, 60), (81_408, 60),
                      (81_409, 60), (3_000, 122), (20_352, 140), (20_353, 140), (40_704, 140),
                      (40_705, 140), (81_409, 140)]}
SLOTS["star_32767"] = lambda: graphgen.star(32_767, 16_000)
SLOTS["star_32768"] = lambda: graphgen.star(32_768, 16_000)
SLOTS["K400"] = lambda: graphgen.complete(400)
SLOTS["hubs"] = lambda: graphgen.rmat(14, 4, seed=5)


def _dev(gs):
    voff = np.cumsum([0] + [g.n for g in gs]).astype(np.int64)
    eoff = np.cumsum([0] + [g.nnz for g in gs]).astype(np.int64)
    rp = np.concatenate([g.rowptr for g in gs]).astype(np.int32)
    ci = np.concatenate([g.colidx for g in gs] + [np.zeros(1, np.int32)]).astype(np.int32)
    return voff, eoff, [torch.from_numpy(x).cuda() for x in (voff, eoff, rp, ci)]


def _check(gc, gs, steps):
    voff, eoff, (v, e, rp, ci) = _dev(gs)
    refs = [oracle.rsc(g.rowptr, g.colidx) for g in gs]
    want = np.concatenate([r.colors for r in refs])
    rounds_want = np.array([r.rounds for r in refs])
    colors, rounds = gc.color_batch(v, e, rp, ci, voff_host=voff, eoff_host=eoff)
    assert np.array_equal(rounds.cpu().numpy(), rounds_want)
    assert np.array_equal(colors.cpu().numpy(), want)
    rows = [(int(voff[i] + i), int(eoff[i]), int(voff[i]), gs[i].n, 0) for i in range(len(gs))]
    for step in steps:
        descs = torch.from_numpy(gc.desc_array(rows).view(np.uint8)).cuda()
        stepped = torch.full((max(int(voff[-1]), 1),), 777, dtype=torch.int32, device="cuda")
        for _ in range(-(-int(rounds_want.max()) // step) + 1):
            gc.batch_step(descs, rp, ci, stepped, step)
            torch.cuda.synchronize()
        d = descs.cpu().numpy().view(gc.DESC_DTYPE)
        assert not d["active"].any()
        assert np.array_equal(d["rounds"], rounds_want)
        assert np.array_equal(stepped.cpu().numpy()[:int(voff[-1])], want)
        assert np.array_equal(d["max_degree"], [int(np.diff(g.rowptr).max(initial=0)) for g in gs])


@pytest.mark.parametrize("name", sorted(SLOTS))
def test_slot_layouts(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] slots {name}", flush=True)
    g = SLOTS[name]()
    # beside graphs that set the launch's length, so that none gets a team
    _check(gc, [graphgen.er(500, 900, 1), g, graphgen.path(70)], [3, 20])


def _tiny(count, seed):
    rng = np.random.default_rng(seed)
    kinds = [graphgen.empty(0), graphgen.empty(1), graphgen.path(2), graphgen.path(65),
             graphgen.complete(30), graphgen.complete(128), graphgen.complete(129),
             graphgen.complete(250), graphgen.star(300, 7), graphgen.er(4095, 9000, 1),
             graphgen.er(4096, 30_719, 2), graphgen.er(64, 300, 3), graphgen.er(100, 300, 4),
             graphgen.er(500, 2000, 5), graphgen.crown(20), _with_clique(2000, 140, 6)]
    return [kinds[i] for i in rng.integers(0, len(kinds), count)]


@pytest.mark.parametrize("extra", ["none", "n4097", "work", "one_60k", "many_large"])
def test_many_small_graphs(extra):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] many small graphs, beside them: {extra}", flush=True)
    more = {"none": [], "n4097": [graphgen.er(4097, 9000, 7)],
            "work": [graphgen.er(4096, 30_720, 8)],  # work 2^16 + 1
            "one_60k": [graphgen.er(60_000, 60_000, 9)],
            "many_large": [graphgen.er(30_000, 200_000, i) for i in range(12)]}[extra]
    gs = _tiny(1100, 11) + more
    _check(gc, gs, [5])
