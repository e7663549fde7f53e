"""GPU parity of the wavefront packing where partitions fill two whole batches
of rounds (961..1024 values, 8-byte columns), whose code has no smaller last
batch: every length of the column's own last partition class, and capacities
that end inside a partition's words.  Bytes equal the oracle's."""
from __future__ import annotations

import os

import numpy as np
import pytest

import paper_2306_15374_amd as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def codec():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    old = os.environ.get("LECO_ENCODE_FUSED_WAVE")
    os.environ["LECO_ENCODE_FUSED_WAVE"] = "0"  # two passes at every size
    try:
        c = P.Codec(0)
    finally:
        if old is None:
            del os.environ["LECO_ENCODE_FUSED_WAVE"]
        else:
            os.environ["LECO_ENCODE_FUSED_WAVE"] = old
    yield c
    c.close()


@pytest.mark.parametrize("L", [960, 961, 1000, 1023, 1024])
@pytest.mark.parametrize("rest", [0, 1, 63, 65, 128, 129, 256, 300, 511, 512, 513, 900])
@pytest.mark.parametrize("dtype", [np.uint32, np.uint64])
def test_last_partition(codec, ref, L, rest, dtype):
    import torch
    rng = np.random.default_rng(L + rest)
    n = 9 * L + min(rest, L - 1)
    bits = rng.integers(0, 8 * np.dtype(dtype).itemsize + 1, 10)
    col = np.concatenate([rng.integers(0, 1 << int(b), L, dtype=np.uint64) if b < 64 else
                          rng.integers(0, (1 << 64) - 1, L, dtype=np.uint64, endpoint=True) for b in bits])[:n]
    col = col.astype(dtype)
    d = torch.from_numpy(col).cuda()
    print(f"[pack] L={L} n={n} {np.dtype(dtype)}", flush=True)
    for reg in ("ls", "minimax", "poly"):
        got = codec.encode(d, fixed_len=L, regressor=reg)
        assert np.array_equal(got.cpu().numpy(), ref.encode(col, fixed_len=L, regressor=reg))


def test_capacity_inside_the_words(codec, ref):
    """A blob that does not fit: LECO_ENOSPC, and nothing written past it."""
    import torch
    rng = np.random.default_rng(5)
    col = rng.integers(0, 1 << 40, 5000, dtype=np.uint64)
    whole = len(ref.encode(col, fixed_len=1000))
    d = torch.from_numpy(col).cuda()
    part, _ = P.make_partitioning(1000)
    for cap in (whole - 16, whole - 5000, 1024):
        buf = torch.full((whole + 4096,), 77, dtype=torch.uint8, device="cuda")
        st, _ = P.leco_encode(codec.ctx, d, len(col), 8, part, buf, cap)
        assert st == P.LECO_ENOSPC
        assert (buf[cap:].cpu().numpy() == 77).all()
