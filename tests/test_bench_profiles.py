"""The benchmark uses a committed traffic summary only while every file that the kernels are made
from is the one it was taken on."""
from __future__ import annotations

import os
import shutil

import pytest

import bench


@pytest.mark.parametrize("name", ["pic_kernels.hip", "pic_runs.h", "pic_device.h", "pic_alt.hip", "pic_internal.h"])
def test_traffic_summary_goes_with_all_kernel_sources(tmp_path, monkeypatch, name):
    csrc, profiles = tmp_path / "csrc", tmp_path / "profiles"
    shutil.copytree(bench.CSRC, csrc)
    profiles.mkdir()
    monkeypatch.setattr(bench, "CSRC", str(csrc))
    monkeypatch.setattr(bench, "PROFILES", str(profiles))
    (profiles / "k_particles_foil_mixed_8x4_traffic.md").write_text(
        f"- hbm_bytes_per_launch: 123\n- kernel_sources_sha256: `{bench.kernel_sources_sha256()}`\n")
    assert bench.measured_traffic("foil", "mixed", (8, 4)) == 123.0
    with open(os.path.join(csrc, name), "a") as f:
        f.write("// changed\n")
    assert bench.measured_traffic("foil", "mixed", (8, 4)) is None
