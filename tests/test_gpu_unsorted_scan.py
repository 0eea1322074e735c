"""GPU: the conflict scans of unsorted rows by a lane (eight entries a step) and by
a group of lanes (four entries per lane a step): row lengths around their steps,
chunks with few and many uncoloured vertices, both algorithms, all light vertices
(a high light / medium split).  Exact equality with the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = {
    # complete graphs: every row has n - 1 entries, one vertex commits per round
    "K8": lambda: graphgen.complete(8),
    "K9": lambda: graphgen.complete(9),
    "K10": lambda: graphgen.complete(10),
    "K65": lambda: graphgen.complete(65),
    "K130": lambda: graphgen.complete(130),
    "star": lambda: graphgen.star(150, 75),
    "er_7": lambda: graphgen.er(1000, 3500, 1),
    "er_16": lambda: graphgen.er(1025, 8200, 2),
    "er_40": lambda: graphgen.er(30_001, 600_000, 3),
}


@pytest.mark.parametrize("algorithm", ["push", "pull"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_unsorted_scans_match_oracle(name, algorithm):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    g = CASES[name]()
    ref = oracle.rsc(g.rowptr, g.colidx)
    h = graphgen.shuffle_rows(g, np.random.default_rng(6))
    for rp64 in (False, True):
        print(f"[case] unsorted {name} {algorithm} rp64={rp64}", flush=True)
        rp = torch.from_numpy(h.rowptr.astype(np.int64 if rp64 else np.int32)).cuda()
        ci = torch.from_numpy(h.colidx).cuda()
        with gc.Graph(rp, ci, rows_sorted=False, algorithm=algorithm, mode="chunked",
                      medium_degree=1000) as G:
            for _ in range(2):
                out = G.color()
                assert G.stats() == (ref.rounds, int(ref.colors.max()) + 1)
                assert np.array_equal(out.cpu().numpy(), ref.colors)
