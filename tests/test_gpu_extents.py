"""GPU round trips of views near the accepted extents.

The oracle would take hours on them, so each band's last columns (or rows) are
compared with the oracle's on that end of the view alone, away from the cut,
and the whole buffer comes back.
"""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

import paper_1803_04880_amd as dwtfrag  # noqa: E402
from oracle import dwt53  # noqa: E402
from paper_1803_04880_amd import learned  # noqa: E402

DEV = "cuda:0"


def _bands(ll, pub, h, w, levels):
    """[(level, band matrix)] of the plain LL and the public fragment."""
    shapes = dwt53.level_shapes(h, w, levels)
    out, off = [(levels, ll.view(shapes[-1]))], 0
    for lv in range(levels, 0, -1):
        (h0, w0), (h1, w1) = shapes[lv - 1], shapes[lv]
        for rows, cols in ((h1, w0 - w1), (h0 - h1, w1), (h0 - h1, w0 - w1)):
            out.append((lv, pub[off:off + rows * cols].view(rows, cols)))
            off += rows * cols
    assert off == pub.numel()
    return out


def _check_end(n, width, levels, axis):
    """Round trip, and the last `keep` samples along `axis` of every band."""
    height = -(-n // width)
    print(f"n={n} width={width} levels={levels}", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n)
    x = torch.randint(0, 256, (n,), generator=gen, device=DEV, dtype=torch.uint8)
    key, nonce = bytes(range(16)), bytes(range(100, 116))
    priv, pub = dwtfrag.protect(x, width, levels, key, nonce)
    back = dwtfrag.restore(priv, pub, n, width, levels, key, nonce)
    assert torch.equal(back, x)
    del back
    # the view's end as the oracle sees it: from a multiple of 2^levels
    size = width if axis else height
    start = (size - 4000) // 64 * 64
    first = start * (1 if axis else width)
    mat = np.zeros((height, size - start) if axis else (size - start, width), np.uint8)
    for r in range(mat.shape[0]):
        a = first + r * width
        row = x[a:min(a + mat.shape[1], r * width + width if axis else n, n)].cpu().numpy()
        mat[r, :row.size] = row
    oll, odet = dwt53.fwd_multilevel(mat, levels)
    want = [oll] + [b for lv in reversed(odet) for b in lv]
    got = _bands(dwtfrag.aes128_ctr(priv, key, nonce).view(torch.int16), pub, height, width, levels)
    keep = 200
    for (lv, g), o in zip(got, want):
        k = min(keep, o.shape[axis])
        a = g.narrow(axis, g.shape[axis] - k, k).cpu().numpy()
        b = o[:, o.shape[1] - k:] if axis else o[o.shape[0] - k:]
        assert np.array_equal(a, b), f"level {lv}"


@pytest.mark.parametrize("levels", [1, 3, 4])
def test_one_row_of_more_than_2_to_28_columns(levels):
    n = (1 << 28) + 1003
    _check_end(n, n, levels, 1)


@pytest.mark.parametrize("levels", [1, 3, 4])
def test_partial_last_row_of_more_than_2_to_28_columns(levels):
    width = (1 << 28) + 4096
    _check_end(2 * width - 5, width, levels, 1)


@pytest.mark.parametrize("levels", [1, 3])
def test_one_column_of_more_rows_than_a_grid_of_short_segments_takes(levels):
    _check_end(1_700_000_000, 1, levels, 0)


def test_learned_column_of_more_tiles_than_a_grid_takes_at_8_wavefronts():
    """2^23 tiles of 32 rows and more; the bytes come back."""
    n = 300_000_001
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n)
    x = torch.randint(0, 256, (n,), generator=gen, device=DEV, dtype=torch.uint8)
    rng = np.random.default_rng(n)
    net = learned.Predictor.from_arrays(rng.integers(-40, 41, (16, 8)), rng.integers(0, 400, 16),
                                        rng.integers(-40, 41, 16), 100, 12)
    print(f"n={n} width=1 learned", flush=True)
    priv, pub = learned.protect(x, 1, 1, bytes(16), bytes(16), net)
    assert torch.equal(learned.restore(priv, pub, n, 1, 1, bytes(16), bytes(16), net), x)


@pytest.mark.parametrize("levels", [0, 5, -1])
def test_tuning_a_depth_that_batches_do_not_have_is_refused(levels):
    from paper_1803_04880_amd import batch
    x = torch.zeros(1000, dtype=torch.uint8, device=DEV)
    with pytest.raises(dwtfrag.DwtfragError):
        batch.tune_classes([x], [32], [levels], trials=1)
