"""Partitions of few values: the fits take the fewest values per lane that
hold a partition and the packing the smallest batch for its last rounds.
Lengths around each step, narrow and wide ranges, every regressor, one-pass
and two-pass sizes, and variable partitions that mix the steps.  Bytes equal
the oracle's."""
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


def column(n, dtype, top, seed):
    rng = np.random.default_rng(seed)
    t = np.arange(n, dtype=np.uint64)
    v = (t % np.uint64(3000)) * np.uint64(max(1, top >> 12))
    return (v + rng.integers(0, max(2, top >> 3), n, dtype=np.uint64)).astype(dtype)


@pytest.mark.parametrize("regressor", ["ls", "minimax", "poly"])
@pytest.mark.parametrize("dtype,top", [(np.uint32, 1 << 16), (np.uint32, 1 << 31), (np.uint64, 1 << 20),
                                       (np.uint64, 1 << 50)])
def test_steps_of_length(codec, ref, regressor, dtype, top):
    import torch
    print(f"[short] {regressor} {np.dtype(dtype)} {top}", flush=True)
    for L in (2, 33, 64, 65, 127, 128, 129, 192, 193, 256, 257, 320, 384, 511, 512, 513, 1024, 1025, 2048):
        for m in (3, 2100) if L <= 128 else (3, 11):
            col = column(m * L - L // 3, dtype, top, L)
            got = codec.encode(torch.from_numpy(col).cuda(), fixed_len=L, regressor=regressor)
            assert np.array_equal(got.cpu().numpy(), ref.encode(col, fixed_len=L, regressor=regressor)), (L, m)
            assert np.array_equal(codec.decode_all(got).cpu().numpy(), col)


@pytest.mark.parametrize("dtype", [np.uint32, np.uint64])
def test_mixed_lengths(codec, ref, dtype):
    import torch
    rng = np.random.default_rng(7)
    lens = rng.choice([1, 2, 64, 65, 128, 129, 250, 256, 257, 512, 513, 1000, 1024], 700)
    starts = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    col = column(int(starts[-1]), dtype, 1 << 18, 9)
    got = codec.encode(torch.from_numpy(col).cuda(), starts=starts)
    assert np.array_equal(got.cpu().numpy(), ref.encode(col, starts=starts))


@pytest.mark.parametrize("regressor", ["ls", "minimax", "poly"])
@pytest.mark.parametrize("dtype,top", [(np.uint32, 1 << 16), (np.uint64, 1 << 40), (np.uint64, 1 << 63)])
def test_many_short(codec, ref, regressor, dtype, top):
    """Enough partitions for several to a wavefront, lengths at the limits of
    that packing, and last partitions of one value and of all but one."""
    import torch
    for L in (31, 32, 33, 64, 100, 127, 170, 171, 255, 256, 257):
        for rest in (1, L - 1):
            n = L * ((1024 if L <= 128 else 4096) * max(1, 512 // L) + 3) + rest
            col = column(n, dtype, top, L)
            print(f"[short] many {regressor} {np.dtype(dtype)} L={L} n={n}", flush=True)
            got = codec.encode(torch.from_numpy(col).cuda(), fixed_len=L, regressor=regressor)
            assert np.array_equal(got.cpu().numpy(), ref.encode(col, fixed_len=L, regressor=regressor)), (L, n)
