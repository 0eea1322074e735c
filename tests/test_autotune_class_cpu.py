"""A tuned setting is kept per algorithm: sequential First Fit and the p-block
colouring, whose times hardly depend on it, must not stand in for the pulled one."""
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")

from paper_1509_08267_amd import autotune, gc  # noqa: E402


def _graph(algorithm):
    options = {gc.GC_OPT_ALGORITHM: gc.ALGORITHMS[algorithm], gc.GC_OPT_MAX_DEGREE: 60}
    return SimpleNamespace(n=1 << 20, m=1 << 25, rowptr=torch.zeros(1, dtype=torch.int32),
                           get=options.__getitem__)


def test_classes_differ_by_algorithm():
    keys = {a: autotune._class_of(_graph(a)) for a in ("push", "pull", "seq", "blocks")}
    assert keys == {a: f"rp32-n20-avg5-max5-{a}" for a in keys}
