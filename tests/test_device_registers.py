"""A kernel that draws through mtgp_device.h and little else keeps eight waves
per SIMD: at most 64 vector registers, and scalar ones that, with the 16 the
trap handler takes, fit an eighth of the SIMD's 800 in blocks of 16."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_eight_waves_per_simd(tmp_path):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", os.path.join(ROOT, "include"), "-Rpass-analysis=kernel-resource-usage",
                        "--offload-device-only", "-S",
                        os.path.join(ROOT, "tests", "shims", "device_draw.hip"),
                        "-o", str(tmp_path / "draw.s")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def count(what):
        return int(re.search(r"%s: (\d+)" % re.escape(what), r.stderr).group(1))

    assert count("SGPRs Spill") == 0 and count("VGPRs Spill") == 0
    assert count("VGPRs") <= 64
    assert (count("TotalSGPRs") + 16 + 15) // 16 * 16 <= 800 // 8
