"""GPU parity of partial last rows at four levels: rows of whole lanes, the
last one ending in the first lane, at and around a lane's boundary and in the
last lane, in one window and in several, behind one and several segments."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

import paper_1803_04880_amd as dwtfrag  # noqa: E402
from oracle import fragment  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("width", [16, 128, 1024, 2400])
@pytest.mark.parametrize("height", [17, 18, 31, 32, 33, 49, 65, 97])
def test_four_levels(width, height):
    for levels in (4, 6):
        for rest in sorted({1, 15, 16, 17, width - 16, width - 1}):
            if not 0 < rest < width:
                continue
            n = (height - 1) * width + rest
            rng = np.random.default_rng([n, levels])
            buf = rng.integers(0, 256, n, dtype=np.uint8)
            key, nonce = rng.bytes(16), rng.bytes(16)
            print(f"n={n} width={width} levels={levels}", flush=True)
            x = torch.from_numpy(buf).to(DEV)
            priv, pub = dwtfrag.protect(x, width, levels, key, nonce)
            out = dwtfrag.restore(priv, pub, n, width, levels, key, nonce)
            opriv, opub = fragment.protect(buf, width, levels, key, nonce)
            assert priv.cpu().numpy().tobytes() == opriv
            assert pub.cpu().numpy().tobytes() == opub
            assert out.cpu().numpy().tobytes() == buf.tobytes()
