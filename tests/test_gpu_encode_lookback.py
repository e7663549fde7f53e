"""One-pass encoders whose wavefronts take their partition by its index: with
no reads of a late predecessor's state allowed they count it themselves, with
the usual number they nearly never do.  Ranges around the narrow fit's limit
at the lengths where its sums are largest, values whose high halves differ,
and residuals too wide for the packing buffer.  Bytes equal the oracle's."""
from __future__ import annotations

import os

import numpy as np
import pytest

import paper_2306_15374_amd as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=["0", "256"])
def codec(request):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    keys = {"LECO_ENCODE_FUSED": "1", "LECO_ENCODE_FUSED_WAVE": "1", "LECO_LOOKBACK_POLLS": request.param}
    old = {k: os.environ.get(k) for k in keys}
    os.environ.update(keys)  # read when the context is created
    try:
        c = P.Codec(0)
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v
    yield c
    c.close()


def shapes(L, top, seed):
    rng = np.random.default_rng(seed)
    t = np.arange(L, dtype=np.uint64)
    r = np.uint64(top)
    parts = [
        rng.integers(0, top + 1, L, dtype=np.uint64),
        np.where(t < L // 2, np.uint64(0), r),          # a step
        np.where(t < L - 1, r, np.uint64(0)),           # the largest sums
        (t % np.uint64(2)) * r,
        (t * r) // np.uint64(max(L - 1, 1)),            # a line through the whole range
        r - (t * r) // np.uint64(max(L - 1, 1)),
    ]
    for p in parts:
        p[0 if p[0] == 0 else -1] = 0
        if p.max() != r:
            p[L // 2] = r
    return np.concatenate(parts * 3 + [parts[0][: L // 2 + 1]])


@pytest.mark.parametrize("L", [2, 3, 64, 1000, 1024, 2049, 4000, 4095, 4096])
@pytest.mark.parametrize("top", [1, (1 << 30) - 1, 1 << 30, (1 << 32) - 1])
def test_ranges(codec, ref, L, top):
    import torch
    base = shapes(L, top, L + top)
    cols = [base.astype(np.uint32), base + np.uint64((1 << 32) - 3), base + np.uint64(1 << 50)]
    for col in cols:
        print(f"[look-back] L={L} top={top} {col.dtype}", flush=True)
        got = codec.encode(torch.from_numpy(col).cuda(), fixed_len=L)
        assert np.array_equal(got.cpu().numpy(), ref.encode(col, fixed_len=L))


@pytest.mark.parametrize("L", [1024, 3000, 4096])
@pytest.mark.parametrize("bits", [60, 61, 62, 63, 64])
def test_wide(codec, ref, L, bits):
    import torch
    rng = np.random.default_rng(bits)
    col = rng.integers(0, (1 << bits) - 1, 9 * L + 100, dtype=np.uint64, endpoint=True)
    print(f"[look-back] L={L} bits={bits}", flush=True)
    got = codec.encode(torch.from_numpy(col).cuda(), fixed_len=L)
    assert np.array_equal(got.cpu().numpy(), ref.encode(col, fixed_len=L))


def test_many(codec, ref):
    import torch
    rng = np.random.default_rng(1)
    for L, n in ((33, 1_500_000), (1024, 6_000_000), (4096, 8_000_000)):
        col = np.cumsum(rng.integers(1, 90, n)).astype(np.uint64)
        print(f"[look-back] many L={L} n={n}", flush=True)
        got = codec.encode(torch.from_numpy(col).cuda(), fixed_len=L)
        assert np.array_equal(got.cpu().numpy(), ref.encode(col, fixed_len=L))
