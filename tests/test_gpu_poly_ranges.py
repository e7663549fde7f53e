"""GPU parity of the polynomial fit where it changes its arithmetic or its
kernel: ranges either side of 2^28 (binary64 sums and residuals below), the
largest residuals that the narrow fit can meet, and lengths around each
kernel's largest.  Bytes equal the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import paper_2306_15374_amd as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def codec():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = P.Codec(0)
    yield c
    c.close()


def shapes(L, top, seed):
    """Partitions of L values whose range is exactly `top`."""
    rng = np.random.default_rng(seed)
    x = np.linspace(-1.0, 1.0, L)
    t = np.arange(L)
    cubic = x**3 - 0.7 * x
    parts = [
        rng.integers(0, top + 1, L),                                  # noise
        (cubic - cubic.min()) / np.ptp(cubic) * top * 0.99,           # a cubic
        t % 2 * top,                                                  # the extremes, alternating
        (t < L // 2) * top,                                           # a step
        (t >= L - 1) * top,                                           # a spike at the end
        (t < 1) * top,                                                # and at the start
        (x * x) * top,
    ]
    out = []
    for p in parts:
        p = np.clip(np.asarray(p, dtype=np.float64).astype(np.int64), 0, top)
        lo, hi = int(np.argmin(p)), int(np.argmax(p))
        if lo == hi:
            hi = (lo + 1) % L
        p[lo], p[hi] = 0, top
        out.append(p)
    return np.concatenate(out + [out[0][: L // 2 + 1]])


@pytest.mark.parametrize("L", [3, 4, 5, 63, 64, 65, 1000, 1023, 1024, 1025, 2000, 2048, 2049, 4095, 4096])
@pytest.mark.parametrize("top", [1, 1000, (1 << 28) - 1, 1 << 28])
def test_range_limit_and_lengths(codec, ref, L, top):
    import torch
    print(f"[poly ranges] L={L} range={top}", flush=True)
    base = shapes(L, top, L + top)
    for col in (base.astype(np.uint32), base.astype(np.uint64) + np.uint64(1 << 40)):
        got = codec.encode(torch.from_numpy(col).cuda(), fixed_len=L, regressor="poly")
        assert np.array_equal(got.cpu().numpy(), ref.encode(col, fixed_len=L, regressor="poly"))
        assert np.array_equal(codec.decode_all(got).cpu().numpy(), col)
