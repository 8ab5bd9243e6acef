"""bench.py reports a profile's HBM bytes only while every source that determines the
launch (kernel, helpers, grid and windows, choice of levels) is the one profiled."""
import hashlib
import json
import os
import shutil

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = "paper_2505_02041_amd/csrc/"
SOURCES = [CSRC + f for f in ("hrc_fused.h", "hrc_kernels.hip", "hrc_api.cpp", "hrc_internal.h")]


@pytest.fixture
def tree(tmp_path, monkeypatch):
    os.makedirs(tmp_path / CSRC)
    os.makedirs(tmp_path / "profiles")
    sha = {}
    for s in SOURCES:
        shutil.copy(os.path.join(ROOT, s), tmp_path / s)
        sha[s] = hashlib.sha256((tmp_path / s).read_bytes()).hexdigest()
    (tmp_path / "profiles" / "hrc_forward_1024_traffic.json").write_text(json.dumps(
        {"kernel": "hrc_fuse_down", "traffic_bytes_per_launch": 7.0, "sources_sha256": sha,
         "source": SOURCES[0], "source_sha256": sha[SOURCES[0]]}))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    return tmp_path


def test_profile_of_the_same_sources(tree):
    assert bench.measured_traffic("hrc_fuse_down") == 7.0
    assert bench.measured_traffic("hrc_fuse_top") is None


@pytest.mark.parametrize("source", SOURCES)
def test_none_once_a_source_changed(tree, source):
    with open(tree / source, "a") as f:
        f.write("\n")
    assert bench.measured_traffic("hrc_fuse_down") is None
