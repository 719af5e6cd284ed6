"""The launches that protect and restore plan, over every accepted extent (CPU
only): ``tests/host/launch_limits.cpp`` is built for the host with api.hip, its
launchers replaced by checks of the plan."""
import os
import subprocess

import pytest

from conftest import ROOT

HIPCC = "/opt/rocm/bin/hipcc"
CSRC = os.path.join(ROOT, "paper_1803_04880_amd", "csrc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_planned_launches_are_within_the_grid_and_the_keystream(tmp_path):
    exe = str(tmp_path / "launch_limits")
    build = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                            "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "api.hip"),
                            os.path.join(ROOT, "tests", "host", "launch_limits.cpp"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stdout + build.stderr
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", ROCR_VISIBLE_DEVICES="")
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    assert run.returncode == 0, run.stdout[-4000:] + run.stderr[-4000:]
    assert " 0 failures" in run.stdout
