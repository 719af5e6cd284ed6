"""The launch shapes that the tuners search (CPU only): what runs differs from
candidate to candidate, and the default is one of them."""
import ctypes
import os
import subprocess

import pytest

from conftest import ROOT

pkg = pytest.importorskip("paper_1803_04880_amd")

HIPCC = "/opt/rocm/bin/hipcc"
CSRC = os.path.join(ROOT, "paper_1803_04880_amd", "csrc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_autotune_times_different_launches(tmp_path):
    exe = str(tmp_path / "autotune_shapes")
    build = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                            "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "api.hip"),
                            os.path.join(ROOT, "tests", "host", "autotune_shapes.cpp"), "-o", exe],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stdout + build.stderr
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", ROCR_VISIBLE_DEVICES="")
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120, env=env)
    assert run.returncode == 0, run.stdout[-4000:] + run.stderr[-4000:]
    assert "\n0 failures" in run.stdout


def _plan_bytes(levels, rows):
    """Device bytes of a batch of one tall buffer under a tile height: they
    grow with the number of tiles."""
    from paper_1803_04880_amd.batch import Item, TuneEntry
    L = pkg.lib()
    items = (Item * 1)()
    it = items[0]
    it.in_ = it.out = it.priv = it.pub = 1 << 20
    it.n, it.width, it.levels = 1000 * 64 * 3 * 5 * 49, 1000, levels
    tune = (TuneEntry * 1)()
    tune[0].width, tune[0].levels, tune[0].launch = 1000, levels, pkg.Launch(rows, 16)
    h = ctypes.c_void_p()
    assert L.dwtfrag_batch_create(ctypes.addressof(items), 1, ctypes.addressof(tune), 1, ctypes.byref(h)) == 0
    n = L.dwtfrag_batch_device_bytes(h)
    L.dwtfrag_batch_destroy(h)
    return n


@pytest.mark.parametrize("levels", [1, 2, 3, 4])
def test_tile_heights_are_what_the_planner_makes_of_them(levels):
    if not os.path.exists(pkg.LIB_PATH):
        pytest.skip("libdwtfrag.so not built")
    from paper_1803_04880_amd import batch as B
    by_rows = {}
    for rows in [0, 1, 2, 7, 8, 16, 17, 24, 32, 47, 48, 64, 65, 96, 127, 128, 200, 256, 1000]:
        by_rows.setdefault(B.tile_rows(rows, levels), set()).add(_plan_bytes(levels, rows))
    assert all(len(v) == 1 for v in by_rows.values())
    sizes = [v.pop() for _, v in sorted(by_rows.items())]
    assert all(a > b for a, b in zip(sizes, sizes[1:]))
    assert max(by_rows) == B.MAX_TILE_ROWS[levels]
    assert B.TILE_SHAPES[0][0] == 0 and B.tile_rows(256, levels) in {B.tile_rows(r, levels) for r, _ in B.TILE_SHAPES}
