"""The stored counter traffic of the fused finest pass counts as current only while the
kernel's source and every header it includes are those it was measured on."""
import json
import os
import shutil

import pytest

import bench
from paper_1506_02079_amd import build


@pytest.mark.parametrize("changed", ["mg_kernels.hip", "wave.h", "device.h", "internal.h", "smooth.h"])
def test_traffic_expires_with_any_source(tmp_path, monkeypatch, changed):
    src = tmp_path / "csrc"
    shutil.copytree(build.CSRC, src)
    os.makedirs(tmp_path / "profiles")
    monkeypatch.setattr(build, "CSRC", str(src))
    monkeypatch.setattr(bench, "MG_SRC", str(src / "mg_kernels.hip"))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    stored = tmp_path / "profiles" / "vcycle_fine_traffic.json"
    stored.write_text(json.dumps({"kernel_sources_sha256": bench.fine_kernel_sha256(), "hbm_bytes_per_launch": 5.0}))
    assert bench.traffic_from_profile() == 5.0
    with open(src / changed, "a") as fh:
        fh.write("\n// one line more\n")
    assert bench.traffic_from_profile() is None


def test_stored_traffic_names_its_sources():
    rec = json.load(open(os.path.join(bench.ROOT, "profiles", "vcycle_fine_traffic.json")))
    assert len(rec["kernel_sources_sha256"]) == 64 and rec["hbm_bytes_per_launch"] > 0
