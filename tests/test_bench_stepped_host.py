"""The benchmark's stored share of stepped crossings is reported only while
everything that decides it is unchanged: the walk's sources and the host code
that chooses between the walks and where the tail walk takes over.
"""
import json
import os
import shutil

import pytest

import bench


@pytest.mark.parametrize("changed", ["paper_2312_11448_amd/csrc/api.hip", "paper_2312_11448_amd/csrc/red_bound.hpp",
                                     "paper_2312_11448_amd/csrc/kernels_tiled.hip"])
def test_share_goes_stale_with_its_sources(tmp_path, monkeypatch, changed):
    shutil.copytree(os.path.join(bench.ROOT, "paper_2312_11448_amd", "csrc"), tmp_path / "paper_2312_11448_amd" / "csrc")
    os.makedirs(tmp_path / "profiles")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    row = {"config": "c3", "profile": "doppler", "stepped_share": 0.5}
    row["source_sha256"] = bench.source_hash(bench.STEPPED_SOURCES)
    (tmp_path / "profiles" / "walk_stepped.json").write_text(json.dumps([row]))
    assert bench.stepped_share("c3", "doppler") == 0.5
    assert bench.stepped_share("c3", "voigt") is None and bench.stepped_share("c2", "doppler") is None
    with open(tmp_path / changed, "a") as fh:
        fh.write("// a comment only\n")
    assert bench.stepped_share("c3", "doppler") == 0.5
    with open(tmp_path / changed, "a") as fh:
        fh.write("int changed;\n")
    assert bench.stepped_share("c3", "doppler") is None
