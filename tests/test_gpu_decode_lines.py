"""Decoders that begin their rounds where a cache line of the output does:
outputs at every kind of offset from one, ranges from any position, shares of
a wavefront either side of 8 KB, partitions that start and end anywhere in a
share.  Decoded values are whole numbers: exact, and nothing beside the range
is written."""
from __future__ import annotations

import os

import numpy as np
import pytest

import paper_2306_15374_amd as P

pytestmark = pytest.mark.gpu


# 2^tile values per workgroup: shares of 256, 1024, 2048 and 4096
@pytest.fixture(scope="module", params=["10", "12", "13", "14"])
def codec(request):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    old = os.environ.get("LECO_TILE_LOG2")
    os.environ["LECO_TILE_LOG2"] = request.param  # read when the context is created
    try:
        c = P.Codec(0)
    finally:
        if old is None:
            del os.environ["LECO_TILE_LOG2"]
        else:
            os.environ["LECO_TILE_LOG2"] = old
    yield c
    c.close()


@pytest.mark.parametrize("L", [1, 50, 65, 333, 1000, 1024, 5000])
@pytest.mark.parametrize("dtype,bits", [(np.uint32, 0), (np.uint32, 7), (np.uint32, 20), (np.uint64, 0),
                                        (np.uint64, 7), (np.uint64, 20), (np.uint64, 40)])
def test_offsets(codec, L, dtype, bits):
    import torch
    rng = np.random.default_rng(L + bits)
    n = 70_000
    col = (np.arange(n, dtype=np.uint64) * np.uint64(3) + rng.integers(0, 1 << bits, n, dtype=np.uint64)).astype(dtype)
    print(f"[lines] L={L} {np.dtype(dtype)} bits={bits}", flush=True)
    blob = codec.encode(torch.from_numpy(col).cuda(), fixed_len=L)
    guard = 99
    tt = torch.int32 if dtype == np.uint32 else torch.int64
    for skew in (0, 1, 16, 63, 64, 77):
        for begin, end in ((0, n), (1, n), (13, 40_000), (63, 64), (64, 64 + 63), (8191, 50_001), (n - 1, n)):
            buf = torch.full((n + 256,), guard, dtype=tt, device="cuda")
            codec.check("leco_decode_range", P.leco_decode_range(
                codec.ctx, blob, blob.numel(), begin, end, buf.data_ptr() + skew * buf.element_size()))
            codec.sync()
            got = buf.cpu().numpy().view(dtype)
            assert np.array_equal(got[skew:skew + end - begin], col[begin:end])
            assert (got[:skew] == guard).all() and (got[skew + end - begin:] == guard).all()
