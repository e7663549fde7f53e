"""GPU split against the oracle where it changes its way: partitions around
the 16 values that one lane tries in a row, columns around the 64 starts of a
step, the 1024-value window, the 2048-value sub-chunk and the 2^20-value
segment, runs that never meet the speculative starts (partitions cut by the
cap alone), and thresholds from below any cost to above all.  Starts are whole
numbers: exact."""
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


def check(codec, ref, col, **kw):
    import torch
    print(f"[split] n={len(col)} {col.dtype} {kw}", flush=True)
    got = codec.partition(torch.from_numpy(np.ascontiguousarray(col)).cuda(), **kw)
    assert np.array_equal(got, ref.partition_greedy(col, **kw))


def jumps(n, lens, dtype, seed):
    """Straight pieces of the given lengths in turn, a jump between them."""
    rng = np.random.default_rng(seed)
    out, at, i = [], 1 << 28, 0
    while sum(map(len, out)) < n:
        k = lens[i % len(lens)]
        out.append(at + 3 * np.arange(k))
        at += 3 * k + int(rng.integers(1 << 10, 1 << 16)) * (1 if i % 2 else -1)
        i += 1
    return np.concatenate(out)[:n].astype(dtype)


@pytest.mark.parametrize("lens", [(2,), (3, 5), (15,), (16,), (17,), (18, 2), (40, 3, 16, 17), (63, 64, 65)])
@pytest.mark.parametrize("dtype", [np.uint32, np.uint64])
def test_piece_lengths(codec, ref, lens, dtype):
    for n in (1, 2, 17, 63, 64, 65, 80, 1023, 1025, 2047, 2048, 2049, 2050, 6200):
        check(codec, ref, jumps(n, lens, dtype, n), tau=0.03, max_passes=1)
    check(codec, ref, jumps(9000, lens, dtype, 9), tau=0.1)


@pytest.mark.parametrize("max_len", [1, 2, 15, 16, 17, 18, 64, 1000, 5000])
def test_cap_alone(codec, ref, max_len):
    rng = np.random.default_rng(max_len)
    line = (7 * np.arange(20_000) + 100).astype(np.uint32)
    noisy = (line + rng.integers(0, 50, len(line))).astype(np.uint64)
    for col in (line, noisy):
        check(codec, ref, col, tau=0.5, max_len=max_len, max_passes=1)


@pytest.mark.parametrize("tau", [-1.0, -0.01, 0.0, 0.003, 0.03, 0.3, 1e9])
@pytest.mark.parametrize("dtype", [np.uint32, np.uint64])
def test_thresholds(codec, ref, tau, dtype):
    rng = np.random.default_rng(3)
    bits = 8 * np.dtype(dtype).itemsize
    wide = rng.integers(0, 1 << (bits - 1), 7000, dtype=np.uint64).astype(dtype)
    slow = np.sort(rng.integers(0, 1 << 20, 7000)).astype(dtype)
    for col in (wide, slow):
        check(codec, ref, col, tau=tau, max_passes=1)
        check(codec, ref, col, tau=tau, max_passes=1, start_positions=True)


@pytest.mark.parametrize("max_len", [1000, 1 << 20])
def test_segments(codec, ref, max_len):
    rng = np.random.default_rng(11)
    n = (1 << 21) + 3000
    col = np.sort(rng.integers(0, 1 << 30, n)).astype(np.uint32)
    col[700_000:1_500_000] = 5 * np.arange(800_000) + int(col[700_000])  # no start for long
    check(codec, ref, col, tau=0.03, max_len=max_len, max_passes=1)
