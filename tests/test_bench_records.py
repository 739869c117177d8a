"""bench.py uses the backprojection's counter record only while every source that
forms the kernel is the one it was taken on: the kernel and both its headers."""
import importlib.util
import json
import os
import shutil

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = ("k_backproject_blocked.hip", "blocked_rows.h", "mfma_lds.h")


@pytest.mark.parametrize("changed", (None,) + SOURCES)
def test_record_is_bound_to_the_kernel_and_its_headers(tmp_path, monkeypatch, changed):
    spec = importlib.util.spec_from_file_location("bench_under_test", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    csrc = tmp_path / "paper_2209_08450_amd" / "csrc"
    os.makedirs(csrc)
    os.makedirs(tmp_path / "profiles")
    for name in SOURCES:
        shutil.copy(os.path.join(ROOT, "paper_2209_08450_amd", "csrc", name), csrc / name)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    record = {"kernel_sha": bench.kernel_source_hash(),
              "f16": {"chunk": 256, "n": 2048, "angles": 2048, "bytes_per_launch": 5.0}}
    json.dump(record, open(tmp_path / "profiles" / "traffic_backproject.json", "w"))
    if changed:
        with open(csrc / changed, "a") as f:
            f.write("// changed\n")
    assert bench.load_traffic("f16", 256, 2048, 2048) == (None if changed else 5.0)
