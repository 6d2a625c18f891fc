"""Launch grids on the host: more workgroups than one grid dimension takes."""

from __future__ import annotations

import os
import subprocess

from paper_2606_30709_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_grids_hold_every_workgroup(tmp_path):
    exe = str(tmp_path / "grid_check")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-w",
                    "-I", build.INCLUDE, "-I", build.CSRC,
                    os.path.join(HERE, "grid_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
