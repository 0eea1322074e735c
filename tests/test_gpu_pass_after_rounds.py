"""GPU: the one-launch passes on a handle that learned its round count another way.
The graphs on which such a pass cannot finish (more than 512 colours in the core
pass, rows that don't fit a workgroup of the resident pass) and graphs just
inside, coloured first by each of the other drivers, by profiled calls or by the
default one, then several times by the default one.  Exact equality with the
oracle's (or, for the cliques, the closed form's) colours, rounds and round
sizes on every call."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _uneven():
    # the rows of one workgroup's chunks (0, 64, 128, ...) hold most entries
    n, rng = 20_032, np.random.default_rng(4)
    edges = set()
    for c in range(0, n // 64, 64):
        for v in range(64 * c, 64 * c + 64):
            for u in rng.integers(0, n, 110):
                if u // 64 % 64:
                    edges.add((min(v, int(u)), max(v, int(u))))
    return graphgen.from_edges(n, edges)


CASES = {
    "K512": lambda: graphgen.complete(512),
    "K513": lambda: graphgen.complete(513),
    "uneven": _uneven,
    "er_10k": lambda: graphgen.er(10_000, 100_000, 5),
    "rmat": lambda: graphgen.rmat(15, 16, seed=3),
}


def _color(gc, G, ref, sizes, what):
    out = G.color()
    assert G.stats() == (ref.rounds, int(ref.colors.max()) + 1), what
    assert np.array_equal(out.cpu().numpy(), ref.colors), what
    assert np.array_equal(G.round_sizes(), sizes), what


@pytest.mark.parametrize("first", ["graph", "host", "chunked", "persistent", "profile"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_default_call_after_another_driver(name, first):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    print(f"[case] {name} after {first}", flush=True)
    g = CASES[name]()
    ref = oracle.rsc(g.rowptr, g.colidx)
    sizes = np.cumsum(np.bincount(ref.round_of, minlength=ref.rounds + 1)[::-1])[::-1][1:]
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    with gc.Graph(rp, ci) as G:
        G.set(*(("profile", 1) if first == "profile" else ("mode", first)))
        _color(gc, G, ref, sizes, "first")
        G.set("profile", 0)
        G.set("mode", "graph")
        for i in range(3):
            _color(gc, G, ref, sizes, i)


def test_many_cliques_above_the_core_colours():
    """300 copies of K_513: the core pass could start late (3,900 vertices
    left after round 500), but the colours run out in it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    k, copies = 513, 300
    print("[case] many K513", flush=True)
    j = torch.arange(k, device="cuda", dtype=torch.int32)
    rows = torch.stack([torch.cat([j[:i], j[i + 1:]]) for i in range(k)])
    ci = (rows[None] + k * torch.arange(copies, device="cuda", dtype=torch.int32)[:, None, None])
    ci = ci.reshape(-1).contiguous()
    rp = torch.arange(k * copies + 1, device="cuda", dtype=torch.int64) * (k - 1)
    want = j.repeat(copies)
    with gc.Graph(rp, ci) as G:
        for i in range(4):
            out = G.color()
            assert G.stats() == (k, k), i
            assert torch.equal(out, want), i
            assert np.array_equal(G.round_sizes(), copies * np.arange(k, 0, -1)), i
