"""The backward's list builder on the host: its wavefronts in several orders
between two barriers (an order of the GPU's choosing there), several (batch,
KV head) pairs, more than 64 key chunks, against a plain enumeration."""

from __future__ import annotations

import os
import subprocess

from paper_2606_30709_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_lists_do_not_depend_on_the_wavefronts_order(tmp_path):
    exe = str(tmp_path / "bwd_lists_check")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-w",
                    "-I", build.INCLUDE, "-I", build.CSRC,
                    os.path.join(HERE, "bwd_lists_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
