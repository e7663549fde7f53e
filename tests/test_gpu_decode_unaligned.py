"""Decoders on partitions whose starts are no multiple of 64: the values
before the next multiple are decoded on their own.  Every residual width from
0 to the column's, both signs of the slope, predictions beyond 2^31, lengths
around one and several rounds, whole columns, ranges and batches.  Decoded
values are whole numbers: exact."""
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


def column(L, dtype, seed):
    """One partition of L values per width and slope."""
    rng = np.random.default_rng(seed)
    bits = 8 * np.dtype(dtype).itemsize
    t = np.arange(L, dtype=object)
    out = []
    for w in range(bits + 1):
        for slope in ((0, 5, -3) if bits == 32 else (0, 7, -7, 1 << 30, -(1 << 30))):
            noise = [int(x) for x in rng.integers(0, 1 << 32, L, dtype=np.uint64)]
            noise = [(x * 0x9E3779B97F4A7C15 >> 7) % (1 << w) for x in noise]
            v = [1000 + slope * int(i) + x for i, x in zip(t, noise)]
            low = min(v)
            out += [(x - low if low < 0 else x) % (1 << bits) for x in v]
    return np.array(out + out[: L // 3 + 1], dtype=dtype)


@pytest.mark.parametrize("L", [1, 33, 63, 65, 127, 300, 700, 999])
@pytest.mark.parametrize("dtype", [np.uint32, np.uint64])
def test_every_width(codec, L, dtype):
    import torch
    col = column(L, dtype, L)
    n = len(col)
    print(f"[unaligned] L={L} {np.dtype(dtype)} n={n}", flush=True)
    blob = codec.encode(torch.from_numpy(col).cuda(), fixed_len=L)
    assert np.array_equal(codec.decode_all(blob).cpu().numpy(), col)
    rng = np.random.default_rng(L)
    for _ in range(4):
        b, e = sorted(int(x) for x in rng.integers(0, n + 1, 2))
        assert np.array_equal(codec.decode_range(blob, b, e).cpu().numpy(), col[b:e])
    out = torch.zeros(n, dtype=torch.uint32 if dtype == np.uint32 else torch.uint64, device="cuda")
    sums = torch.zeros(3, dtype=torch.uint64, device="cuda")
    lo, hi = int(col.min()), int(col.max())
    batch = P.leco_batch_create(codec.ctx, [P.DecodeJob(blob.data_ptr(), blob.numel(), n, out.data_ptr(),
                                                        lo, hi, sums.data_ptr())])
    try:
        for op in (P.LECO_BATCH_DECODE, P.LECO_BATCH_DECODE | P.LECO_BATCH_FILTER):
            out.zero_()
            codec.check("leco_batch_run", P.leco_batch_run(batch, op))
            codec.sync()
            assert np.array_equal(out.cpu().numpy(), col)
    finally:
        P.leco_batch_destroy(batch)
