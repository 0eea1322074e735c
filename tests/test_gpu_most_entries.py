"""GPU: 32-bit row pointers up to their end: 2^31 - 2 CSR entries, so that the
position behind the last rows' last steps no longer fits 31 bits (the library then
works on a 64-bit copy of them), and the most entries without one.  Cliques of 65
vertices, single edges, and a clique of 120 vertices whose rows come last: every
driver and degree class that walks rows, and the check of the CSR.  The expected
colours, rounds and round sizes are the cliques' closed form (the p-block
algorithm: a proper colouring)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

K, LAST = 65, 120
SIZES = [2**31 - 2, 2**31 - 8194]


def _parts(m):
    # cliques of K, and single edges that fill up
    pairs = (m - LAST * (LAST - 1)) % (K * (K - 1)) // 2
    return (m - LAST * (LAST - 1) - 2 * pairs) // (K * (K - 1)), pairs


def _clique_rows(k, device):
    j = torch.arange(k, dtype=torch.int32, device=device)
    return torch.stack([torch.cat([j[:i], j[i + 1:]]) for i in range(k)])


@pytest.fixture(scope="module", params=SIZES)
def graph(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = "cuda"
    M = request.param
    Q, PAIRS = _parts(M)
    ci = torch.empty(M, dtype=torch.int32, device=dev)
    rows = _clique_rows(K, dev).reshape(1, -1)
    body = ci[:Q * K * (K - 1)].view(Q, K * (K - 1))
    for a in range(0, Q, 65536):
        b = min(Q, a + 65536)
        base = K * torch.arange(a, b, dtype=torch.int32, device=dev)
        torch.add(rows, base[:, None], out=body[a:b])
    at, v = Q * K * (K - 1), Q * K
    pair = torch.arange(2 * PAIRS, dtype=torch.int32, device=dev) ^ 1
    ci[at:at + 2 * PAIRS] = pair + v
    ci[at + 2 * PAIRS:] = _clique_rows(LAST, dev).reshape(-1) + (v + 2 * PAIRS)
    deg = torch.cat([torch.full((v,), K - 1), torch.ones(2 * PAIRS, dtype=torch.int64),
                     torch.full((LAST,), LAST - 1)]).to(dev)
    rp = torch.zeros(deg.numel() + 1, dtype=torch.int64, device=dev)
    torch.cumsum(deg, 0, out=rp[1:])
    assert int(rp[-1]) == M
    want = torch.cat([torch.arange(K, dtype=torch.int32, device=dev).repeat(Q),
                      torch.arange(2, dtype=torch.int32, device=dev).repeat(PAIRS),
                      torch.arange(LAST, dtype=torch.int32, device=dev)])
    yield rp.to(torch.int32), ci, want


def _sizes(m):
    Q, PAIRS = _parts(m)
    r = np.arange(1, LAST + 1)
    return Q * np.maximum(K + 1 - r, 0) + PAIRS * np.maximum(3 - r, 0) + LAST + 1 - r


@pytest.mark.parametrize("name, sorted_rows, options", [
    ("default", True, {}),
    ("wavefront class", True, {"medium_degree": 100}),
    ("workgroup class", True, {"medium_degree": 100, "heavy_degree": 101}),
    ("pull", True, {"algorithm": "pull"}),
    ("unsorted", False, {}),
    ("unsorted wavefront class", False, {"medium_degree": 100}),
    ("persistent", True, {"mode": "persistent"}),
    ("seq", True, {"algorithm": "seq"}),
    ("seq unsorted", False, {"algorithm": "seq"}),
    ("seq wavefront class", True, {"algorithm": "seq", "medium_degree": 100}),
    ("seq by rounds", True, {"algorithm": "seq", "mode": "host"}),
])
def test_cliques_up_to_the_last_entry(graph, name, sorted_rows, options):
    from paper_1509_08267_amd import gc
    rp, ci, want = graph
    with gc.Graph(rp, ci, rows_sorted=sorted_rows, **options) as G:
        for i in range(2):
            print(f"[case] most entries: {name}, call {i}", flush=True)
            out = G.color()
            assert G.stats() == (LAST, LAST)
            assert torch.equal(out, want)
            assert np.array_equal(G.round_sizes(), _sizes(ci.numel()))


@pytest.mark.parametrize("per_block", [128, 400])  # masks, slots
def test_blocks_up_to_the_last_entry(graph, per_block):
    from paper_1509_08267_amd import gc
    rp, ci, want = graph
    print(f"[case] most entries: blocks of {per_block}", flush=True)
    Q, PAIRS = _parts(ci.numel())
    with gc.Graph(rp, ci, algorithm="blocks", partitions=want.numel() // per_block) as G:
        out = G.color()
        G.stats()
        for lo, count, k in ((0, Q, K), (Q * K, PAIRS, 2), (Q * K + 2 * PAIRS, 1, LAST)):
            c = out[lo:lo + count * k].view(count, k).sort(dim=1).values
            assert int(c.min()) == 0 and bool((c.diff(dim=1) > 0).all())


def test_validation_up_to_the_last_entry(graph):
    from paper_1509_08267_amd import gc
    rp, ci, _ = graph
    print("[case] most entries: validation", flush=True)
    gc.Graph(rp, ci, validate=True).close()
    keep = ci[-1].clone()
    ci[-1] = ci[-2]
    try:
        with pytest.raises(gc.GCError):
            gc.Graph(rp, ci, validate=True)
    finally:
        ci[-1] = keep
