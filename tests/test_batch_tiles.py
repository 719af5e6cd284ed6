"""A batch's tile lists and the time that planning them takes (CPU only):
``tests/host/batch_tiles.cpp`` is built for the host around batch.hip and run."""
import os
import subprocess

import pytest

from conftest import ROOT

HIPCC = "/opt/rocm/bin/hipcc"
CSRC = os.path.join(ROOT, "paper_1803_04880_amd", "csrc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_tile_lists_are_longest_first_and_cheap_to_plan(tmp_path):
    exe = str(tmp_path / "batch_tiles")
    build = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O3", "-std=c++17",
                            "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "api.hip"),
                            os.path.join(ROOT, "tests", "host", "batch_tiles.cpp"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stdout + build.stderr
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", ROCR_VISIBLE_DEVICES="")
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120, env=env)
    assert run.returncode == 0, run.stdout[-4000:] + run.stderr[-4000:]
    assert "\n0 failures" in run.stdout
