"""The index arithmetic at a view's end, up to the widest rows (CPU only):
``tests/host/row_ends.cpp`` is built for the host from the kernels' own header
and run."""
import os
import subprocess

import pytest

from conftest import ROOT

HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_samples_at_the_end_of_a_view(tmp_path):
    exe = str(tmp_path / "row_ends")
    build = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                            "-I", os.path.join(ROOT, "paper_1803_04880_amd", "csrc"),
                            os.path.join(ROOT, "tests", "host", "row_ends.cpp"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stdout + build.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-4000:] + run.stderr[-4000:]
    assert " 0 failures" in run.stdout
