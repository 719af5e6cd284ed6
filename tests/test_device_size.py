"""Launch planning on devices of other sizes than a whole MI355X (CPU only):
``tests/host/device_size.cpp`` is built for the host with api.hip, the device
queries replaced."""
import os
import subprocess

import pytest

from conftest import ROOT

HIPCC = "/opt/rocm/bin/hipcc"
CSRC = os.path.join(ROOT, "paper_1803_04880_amd", "csrc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_segments_follow_the_device_s_compute_units(tmp_path):
    exe = str(tmp_path / "device_size")
    build = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                            "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "api.hip"),
                            os.path.join(ROOT, "tests", "host", "device_size.cpp"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stdout + build.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-4000:] + run.stderr[-4000:]
    assert "\n0 failures" in run.stdout
