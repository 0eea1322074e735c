"""The hash that ties a counter summary to the kernels it was taken on changes with
every source of the library."""
import importlib.util
import os
import shutil

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1509_08267_amd", "csrc")


@pytest.mark.parametrize("name", sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".h"))))
def test_hash_covers_every_source(name, tmp_path, monkeypatch):
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    copy = tmp_path / "paper_1509_08267_amd" / "csrc"
    shutil.copytree(CSRC, copy)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    before = bench.kernel_source_hash()
    with open(copy / name, "a") as f:
        f.write("\n")
    assert bench.kernel_source_hash() != before
