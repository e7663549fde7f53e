"""GPU split against the oracle where values join in whole steps of 64 because
their first differences lie within the partition's own: a difference further
out, an end of the column, the length cap and starting partitions at and
around the steps' edges, and thresholds either side of D~.  Starts are whole
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
    print(f"[steady] n={len(col)} {col.dtype} {kw}", flush=True)
    got = codec.partition(torch.from_numpy(np.ascontiguousarray(col)).cuda(), **kw)
    assert np.array_equal(got, ref.partition_greedy(col, **kw))


@pytest.mark.parametrize("n", [66, 129, 2048, 2049, 2113, 4160, 6200])
@pytest.mark.parametrize("dtype", [np.uint32, np.uint64])
def test_outlier_around_the_edges(codec, ref, n, dtype):
    """Differences of 0 .. 7, one or two of another size."""
    rng = np.random.default_rng(n)
    for at in (1, 2, 63, 64, 65, 66, 127, 128, 129, 2047, 2048, 2049, 2111, n - 1):
        if at >= n:
            continue
        for jump in (-3, 8, 200, 1 << 20):
            d = rng.integers(0, 8, n)
            d[1:3] = (0, 7)
            d[at] = jump
            col = ((1 << 22) + np.cumsum(d)).astype(dtype)
            check(codec, ref, col, tau=0.05, max_passes=1)


@pytest.mark.parametrize("bits", [3, 40, 62])
@pytest.mark.parametrize("over", [-1, 0, 1])
def test_threshold_at_the_width(codec, ref, bits, over):
    """tau S_M one below, at and one above the differences' width."""
    rng = np.random.default_rng(bits)
    top = (1 << bits) - 1
    d = np.tile(np.array([0, top, 0, 0], dtype=np.uint64), 1500)
    d[5:] = np.where(rng.integers(0, 2, len(d) - 5) == 1, np.uint64(top), np.uint64(0))
    alternate = np.cumsum(np.where(np.arange(len(d)) % 2 == 0, d, -d), dtype=np.uint64)
    for col in (np.cumsum(d, dtype=np.uint64), alternate + np.uint64(1 << 63)):
        check(codec, ref, col, tau=1.0, sm_bits=bits + over, max_passes=1)


@pytest.mark.parametrize("cap", [63, 64, 65, 66, 127, 129, 191, 2047, 2050])
def test_cap_within_a_step(codec, ref, cap):
    col = np.full(9000, 77, dtype=np.uint64)
    check(codec, ref, col, tau=0.1, max_len=cap)
    check(codec, ref, col + (np.arange(9000) % 3 == 0).astype(np.uint64), tau=0.1, max_len=cap)
    check(codec, ref, col, tau=0.1, max_len=cap, start_positions=True)


@pytest.mark.parametrize("at", [62, 63, 64, 65, 66, 128, 190, 2046, 2048, 2050])
@pytest.mark.parametrize("length", [3, 64, 70, 200])
def test_starting_partition_within_a_step(codec, ref, at, length):
    """Values whose second differences are never 0 except along one run."""
    n = 4500
    d = np.where(np.arange(n) % 2 == 0, 5, 9)
    d[at:at + length] = 7
    col = (1000 + np.cumsum(d)).astype(np.uint64)
    check(codec, ref, col, tau=0.05, start_positions=True, max_passes=1)
    check(codec, ref, col, tau=0.001, start_positions=True, max_passes=1)
