"""GPU parity of batches on both sides of the rule that picks the kernel whose
plain form takes partial last rows: only whole rows, only partial ones, and a
long drain with a few, at every depth; widths of whole lanes and others."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

import paper_1803_04880_amd as dwtfrag  # noqa: E402
from oracle import fragment  # noqa: E402
from paper_1803_04880_amd import batch as B  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("rest", ["whole", "partial", "one partial"])
@pytest.mark.parametrize("heights", [(1, 2, 7, 16), (17, 49, 96, 131)])
def test_batches_match_the_oracle(rest, heights):
    rng = np.random.default_rng([len(rest), heights[0]])
    specs = []
    for levels in (1, 2, 3, 4):
        for width in (16, 160, 1024, 1040, 2400, 77, 1501):
            for h in heights:
                part = rest == "partial" or (rest == "one partial" and not specs)
                n = h * width - (int(rng.integers(1, width)) if part else 0)
                specs.append((n, width, levels, rng.integers(0, 256, n, dtype=np.uint8), rng.bytes(16), rng.bytes(16)))
    print(f"{len(specs)} items, {rest}, heights {heights}", flush=True)
    xs = [torch.from_numpy(s[3]).to(DEV) for s in specs]
    b = B.Batch(xs, [s[1] for s in specs], [s[2] for s in specs], [s[4] for s in specs], [s[5] for s in specs])
    for _ in range(2):
        b.protect()
        b.restore()
    torch.cuda.synchronize()
    for i, (n, width, levels, buf, key, nonce) in enumerate(specs):
        priv, pub = fragment.protect(buf, width, levels, key, nonce)
        assert b.privs[i].cpu().numpy().tobytes() == priv, (n, width, levels)
        assert b.pubs[i].cpu().numpy().tobytes() == pub, (n, width, levels)
        assert b.outs[i].cpu().numpy().tobytes() == buf.tobytes(), (n, width, levels)


def test_long_drain_with_few_partial_rows():
    """More tiles than a few rounds, a partial row among every hundred: equal
    to lone calls."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7)
    sizes = [(1 << 26, 4096, 1)] * 3 + [(1 << 24, 4096, lv) for lv in (2, 3, 4)] + [((1 << 20) - 5, 1024, lv) for lv in (1, 2, 3, 4)]
    xs = [torch.randint(0, 256, (n,), generator=gen, device=DEV, dtype=torch.uint8) for n, _, _ in sizes]
    key, nonce = bytes(range(16)), bytes(range(50, 66))
    b = B.Batch(xs, [w for _, w, _ in sizes], [lv for _, _, lv in sizes], [key] * len(xs), [nonce] * len(xs))
    b.protect()
    b.restore()
    torch.cuda.synchronize()
    for i, (n, w, lv) in enumerate(sizes):
        print(f"n={n} width={w} levels={lv}", flush=True)
        priv, pub = dwtfrag.protect(xs[i], w, lv, key, nonce)
        assert torch.equal(b.privs[i], priv) and torch.equal(b.pubs[i], pub)
        assert torch.equal(b.outs[i], xs[i])


@pytest.mark.parametrize("tall", [False, True])
def test_batches_of_few_rows_only(tall):
    """Every item has one LL row: kernels of their own; also with values
    outside the packed range in some fragments."""
    rng = np.random.default_rng(23 + tall)
    specs = []
    for levels in (1, 2, 3, 4):
        for width in (1, 2, 5, 16, 160, 1024, 1040, 2400, 77, 1501):
            half, unit = 1 << (levels - 1), 1 << levels
            for h in ((half + 1, unit) if tall and width % 16 else (1, half)):
                n = h * width - (int(rng.integers(0, width)) if len(specs) % 2 else 0)
                n = max(n, (h - 1) * width + 1)
                specs.append((n, width, levels, rng.integers(0, 256, n, dtype=np.uint8), rng.bytes(16), rng.bytes(16)))
    print(f"{len(specs)} items", flush=True)
    xs = [torch.from_numpy(s[3]).to(DEV) for s in specs]
    b = B.Batch(xs, [s[1] for s in specs], [s[2] for s in specs], [s[4] for s in specs], [s[5] for s in specs])
    for _ in range(2):
        b.protect()
        b.restore()
    torch.cuda.synchronize()
    for i, (n, width, levels, buf, key, nonce) in enumerate(specs):
        priv, pub = fragment.protect(buf, width, levels, key, nonce)
        assert b.privs[i].cpu().numpy().tobytes() == priv, (n, width, levels)
        assert b.pubs[i].cpu().numpy().tobytes() == pub, (n, width, levels)
        assert b.outs[i].cpu().numpy().tobytes() == buf.tobytes(), (n, width, levels)
    for i in range(0, len(specs), 3):
        n, width, levels, _, key, nonce = specs[i]
        if b.pubs[i].numel():
            b.pubs[i][rng.integers(0, b.pubs[i].numel())] = 20000
    b.restore()
    torch.cuda.synchronize()
    for i, (n, width, levels, buf, key, nonce) in enumerate(specs):
        want = fragment.restore(b.privs[i].cpu().numpy().tobytes(), b.pubs[i].cpu().numpy().tobytes(), n, width, levels,
                                key, nonce)
        assert b.outs[i].cpu().numpy().tobytes() == want, (n, width, levels)
