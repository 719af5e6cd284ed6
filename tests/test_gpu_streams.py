"""GPU parity of the streaming kernels at the edges of what a wavefront covers.

Widths around a lane's columns, a window's lanes and its owned columns;
heights around the unit of 2^levels rows and a segment's rows; partial last
rows that end inside any of them; every depth of a fused stage at both lane
widths.  Integer work: fragments equal the oracle's byte for byte, and
restore returns the input.
"""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

import paper_1803_04880_amd as dwtfrag  # noqa: E402
from oracle import aes128, fragment  # noqa: E402

DEV = "cuda:0"


def _check(n, width, levels, launch):
    rng = np.random.default_rng([n, width, levels])
    buf = rng.integers(0, 256, n, dtype=np.uint8)
    key, nonce = rng.bytes(16), rng.bytes(16)
    print(f"n={n} width={width} levels={levels} launch={launch}", flush=True)
    x = torch.from_numpy(buf).to(DEV)
    priv, pub = dwtfrag.protect(x, width, levels, key, nonce, launch=launch)
    out = dwtfrag.restore(priv, pub, n, width, levels, key, nonce, launch=launch)
    opriv, opub = fragment.protect(buf, width, levels, key, nonce)
    assert priv.cpu().numpy().tobytes() == opriv
    assert pub.cpu().numpy().tobytes() == opub
    assert out.cpu().numpy().tobytes() == buf.tobytes()


@pytest.mark.parametrize("levels,cols", [(1, 8), (2, 8), (3, 8), (1, 16), (2, 16), (3, 16), (4, 16)])
@pytest.mark.parametrize("span", [1, 4])
def test_window_edges(levels, cols, span):
    """Rows ending at, before and after a lane, a window (64 lanes) and an
    owned range (whole 128-column pieces of it)."""
    if span == 1:
        widths = [1, 2, 3, cols - 1, cols, cols + 1, 2 * cols, 9 * cols + 5]
    else:
        win, own = 64 * cols, (64 * cols - 48) // 128 * 128
        widths = [win - 1, win, win + 1, win + cols, own + 8, 2 * own - 1, 2 * own, 2 * own + 7]
    for i, width in enumerate(widths):
        height = 37 + 5 * i
        _check(height * width - (i % 3) * (width // 3), width, levels, (0, cols))


@pytest.mark.parametrize("levels,cols", [(1, 8), (2, 8), (3, 8), (1, 16), (2, 16), (3, 16), (4, 16)])
def test_segment_edges(levels, cols):
    """Heights around one and two units, and around a segment's rows."""
    unit = 1 << levels
    width = 8 * cols + 3
    for height in sorted({1, 2, unit - 1, unit, unit + 1, 2 * unit - 1, 2 * unit + 1, 4 * unit,
                          4 * unit + 1, 9 * unit - 1, 9 * unit + 2}):
        if height < 1:
            continue
        _check(height * width - (width // 2 if height % 2 else 0), width, levels, (0, cols))
        _check(height * width, width - 3, levels, (4 * unit, cols))


@pytest.mark.parametrize("width", [512, 1000, 1021])
@pytest.mark.parametrize("levels", [1, 2, 3, 4])
def test_partial_last_row(width, levels):
    """The view's last row ends inside the first lane, a window, the last one."""
    for rest in (1, 3, width // 2, width - 1):
        _check(70 * width + rest, width, levels, None)


@pytest.mark.parametrize("levels", [5, 6, 8])
def test_deep_stages(levels):
    """int16 stages behind the byte stage, at odd and even inner sizes."""
    for width, height in ((2064, 530), (1037, 611)):
        _check(width * height - 11, width, levels, None)


@pytest.mark.parametrize("levels,cols", [(1, 8), (2, 8), (3, 8), (1, 16), (2, 16), (3, 16), (4, 16)])
def test_restore_window_edges(levels, cols):
    """Rows ending around the columns that an inverse window owns: at one
    level all but the halos, else whole 64-column pieces."""
    own = 64 * cols - 16 if cols == 8 else 64 * cols - 32
    own = own if levels == 1 else own // 64 * 64
    for i, width in enumerate([own - 1, own, own + 1, own + cols - 1, own + cols, 2 * own, 2 * own + 3]):
        _check((19 + 3 * i) * width - (i % 3) * (width // 3), width, levels, (0, cols))


@pytest.mark.parametrize("width", [1, 2, 5, 19, 77, 501, 1001])
@pytest.mark.parametrize("levels", [1, 2, 3, 4])
def test_values_outside_the_packed_range_at_row_ends(width, levels):
    """Values outside [-4096, 4095] in the last column of a band row, where
    the row's end cuts a lane and the next row's values follow in the
    fragment, and in the fragment's last values: the exact inverse, from each
    alone and from all."""
    height = 45
    n = height * width
    rng = np.random.default_rng([width, levels])
    key, nonce = rng.bytes(16), rng.bytes(16)
    g = fragment.geometry(n, width, levels)
    shapes = g["shapes"]
    ends = []                      # the last value of some row of each band
    off = 0
    for l in range(levels, 0, -1):
        (h0, w0), (h1, w1) = shapes[l - 1], shapes[l]
        for rows, cols in ((h1, w0 - w1), (h0 - h1, w1), (h0 - h1, w0 - w1)):
            if rows * cols:
                ends.append(off + (rows // 2 + 1) * cols - 1 if rows > 1 else off + cols - 1)
            off += rows * cols
    base_ll = rng.integers(-200, 600, g["priv_bytes"] // 2).astype("<i2")
    base_pub = rng.integers(-300, 301, g["pub_bytes"] // 2).astype("<i2")
    last = base_pub.size - 1
    for where in [[e] for e in ends[:3]] + [[last], ends]:
        ll, pub = base_ll.copy(), base_pub.copy()
        for e in where:
            if 0 <= e < pub.size:
                pub[e] = 20000
        if len(where) > 1:
            ll[-1] = -20000
        priv = aes128.ctr_xor(key, nonce, ll.tobytes()).tobytes()
        print(f"width={width} levels={levels} outside at {where}", flush=True)
        tp = torch.from_numpy(np.frombuffer(priv, np.uint8).copy()).to(DEV)
        tq = torch.from_numpy(pub).to(DEV)
        got = dwtfrag.restore(tp, tq, n, width, levels, key, nonce).cpu().numpy().tobytes()
        assert got == fragment.restore(priv, pub.tobytes(), n, width, levels, key, nonce)


@pytest.mark.parametrize("levels,cols", [(1, 8), (2, 8), (3, 8), (1, 16), (2, 16), (3, 16)])
@pytest.mark.parametrize("height", [1, 2, 9, 41])
def test_partial_last_row_of_whole_lanes(levels, cols, height):
    """Rows of whole lanes (no window cuts one), the last row ending in the
    first lane, at and around a lane's boundary, in the last lane; in one
    window and in several."""
    for width in (8 * cols, 64 * cols, 150 * cols):
        for rest in (1, cols - 1, cols, cols + 1, width - cols, width - 1):
            _check((height - 1) * width + rest, width, levels, (0, cols))
