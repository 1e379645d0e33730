"""The sources that the bench's counter profile of the block GEMV is tied to: the kernels, the tile layout
and the wave program that they share with others."""
import hashlib
import importlib.util
import os
import shutil

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = ("kernels_apply.hip", "device_common.h", "tile_gemv.h")


@pytest.mark.parametrize("changed", SOURCES)
def test_profile_is_detached_by_a_change_of_any_source(changed, tmp_path, monkeypatch):
    spec = importlib.util.spec_from_file_location("bench_sources", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    csrc = tmp_path / "paper_2501_17656_amd" / "csrc"
    csrc.mkdir(parents=True)
    h = hashlib.sha256()
    for f in SOURCES:
        shutil.copy(os.path.join(ROOT, "paper_2501_17656_amd", "csrc", f), csrc / f)
        h.update((csrc / f).read_bytes())
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "gemv_counters_test.md").write_text(
        "    traffic gemv_fp64 src=%s per_launch_bytes=3.0e+10 alg_per_launch_bytes=2.0e+10\n" % h.hexdigest()[:16])
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.profiled_traffic("gemv_fp64", 4.0e9) == round(6.0e9)
    with open(csrc / changed, "a") as f:
        f.write("\n// changed\n")
    assert bench.profiled_traffic("gemv_fp64", 4.0e9) is None
