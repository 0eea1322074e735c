"""GPU: calls that make graphs of their rounds in two threads while others wait for the
whole device: the calls give their results, and no wait is refused."""
import threading
import time

import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_graphs_of_rounds_beside_device_waits():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1509_08267_amd import gc
    cases = []
    for g in (graphgen.er(60_000, 200_000, 5), graphgen.rmat(15, 8, seed=2)):
        cases.append((torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda(),
                      oracle.rsc(g.rowptr, g.colidx)))
    torch.cuda.synchronize()
    end = time.monotonic() + 3
    failed, calls = [], [0, 0]

    def color(i):
        rp, ci, ref = cases[i]
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                while time.monotonic() < end:
                    with gc.Graph(rp, ci) as G:
                        for lanes in (4, 8):
                            G.set("lanes", lanes)
                            for _ in range(2):
                                out = G.color()
                                assert G.stats()[0] == ref.rounds
                        assert np.array_equal(out.cpu().numpy(), ref.colors)
                    calls[i] += 1
        except BaseException as e:  # noqa: BLE001
            failed.append(repr(e))

    def wait():
        while time.monotonic() < end:
            try:
                torch.cuda.synchronize()
            except BaseException as e:  # noqa: BLE001
                failed.append(repr(e))
                return
            time.sleep(0.0002)

    threads = [threading.Thread(target=color, args=(i,)) for i in (0, 1)]
    threads += [threading.Thread(target=wait) for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
    assert min(calls) > 3
