"""GPU parity of views of few rows: every height up to past one unit of
2^levels rows, where the kernels change, at widths around a lane's columns and
a window's; partial last rows; inner stages of few rows; fragments with values
outside the packed range.  Byte for byte against the oracle."""
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
SHAPES = [(1, 8), (2, 8), (3, 8), (1, 16), (2, 16), (3, 16), (4, 16)]


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


@pytest.mark.parametrize("levels,cols", SHAPES)
@pytest.mark.parametrize("height", list(range(1, 19)))
def test_heights_up_to_a_unit(levels, cols, height):
    if height > (1 << levels) + 2:
        pytest.skip("past the unit")
    for width in (1, 2, 3, cols - 1, cols, cols + 1, 5 * cols + 3, 64 * cols, 64 * cols + cols, 150 * cols - 5):
        full = height * width
        for n in {full, full - width // 2, full - width + 1}:
            if n > (height - 1) * width:
                _check(n, width, levels, (0, cols))


@pytest.mark.parametrize("levels", [5, 6, 7, 8])
@pytest.mark.parametrize("height", [1, 2, 3, 15, 16, 17, 33, 100, 129])
def test_inner_stages_of_few_rows(levels, height):
    for width in (37, 600, 4096):
        _check(height * width - width // 3, width, levels, None)


@pytest.mark.parametrize("levels,cols", SHAPES)
@pytest.mark.parametrize("width", [1, 2, 5, 16, 77, 1001, 2048])
def test_values_outside_the_packed_range(levels, cols, width):
    """One such value in turn in each band, and many: the exact inverse."""
    for height in {1, 2, (1 << levels) - 1, 1 << levels} - {0}:
        n = height * width
        rng = np.random.default_rng([width, levels, height])
        key, nonce = rng.bytes(16), rng.bytes(16)
        g = fragment.geometry(n, width, levels)
        base_ll = rng.integers(-200, 600, g["priv_bytes"] // 2).astype("<i2")
        base_pub = rng.integers(-300, 301, g["pub_bytes"] // 2).astype("<i2")
        size = base_pub.size
        spots = sorted({0, size // 3, size // 2, size - 1}) if size else []
        for where in [[s] for s in spots] + [spots]:
            ll, pub = base_ll.copy(), base_pub.copy()
            for s in where:
                pub[s] = 20000
            if len(where) != 1:
                ll[-1] = -20000
            priv = aes128.ctr_xor(key, nonce, ll.tobytes()).tobytes()
            print(f"width={width} levels={levels} height={height} outside at {where}", flush=True)
            got = dwtfrag.restore(torch.from_numpy(np.frombuffer(priv, np.uint8).copy()).to(DEV),
                                  torch.from_numpy(pub).to(DEV), n, width, levels, key, nonce, launch=(0, cols))
            assert got.cpu().numpy().tobytes() == fragment.restore(priv, pub.tobytes(), n, width, levels, key, nonce)
