"""GPU merge scan against the oracle where its workgroup walk changes its
way of sizing a union: batches and windows of 256 partitions, chunks of 1024,
neighbours sized one at a time (over 256 values, over 8192 with hulls), hulls
built after eight such merges, hulls that outgrow 64 vertices, and unions at
the cap.  Starts are whole numbers: exact."""
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
    print(f"[merge] n={len(col)} {col.dtype} {kw}", flush=True)
    got = codec.partition(torch.from_numpy(np.ascontiguousarray(col)).cuda(), **kw)
    assert np.array_equal(got, ref.partition_greedy(col, **kw))
    return len(got) - 1


def steps(lens, slope, noise, seed, jump):
    """Lines of the given lengths, each `jump` off the one before, with
    noise U{0..noise-1}: the split cuts at every jump."""
    rng = np.random.default_rng(seed)
    v, level = [], 1 << 20
    for i, n in enumerate(lens):
        v.append(level + slope * np.arange(n) + rng.integers(0, noise, n))
        level += slope * n + (jump if i % 2 else -jump)
    return np.concatenate(v).astype(np.uint64)


@pytest.mark.parametrize("n", [509, 512, 515, 1021, 1027, 2045, 2051, 4090, 4100, 8190])
@pytest.mark.parametrize("dtype", [np.uint32, np.uint64])
def test_batch_window_and_chunk_edges(codec, ref, n, dtype):
    """tau = 0 leaves partitions of about two values, so batches, windows and
    chunks end all around these lengths."""
    rng = np.random.default_rng(n)
    col = (np.arange(n) * 11 + rng.integers(0, 256, n) + 5000).astype(dtype)
    check(codec, ref, col, tau=0.0)
    check(codec, ref, col, tau=0.0, max_passes=1, max_len=300)


@pytest.mark.parametrize("piece", [200, 256, 257, 400, 3000])
@pytest.mark.parametrize("shift", [0, 30])
def test_long_neighbours(codec, ref, piece, shift):
    """Pieces either side of the one-at-a-time length, small jumps (merged
    across) between them; shifted values take the 64- and 128-bit turns."""
    rng = np.random.default_rng(piece)
    lens = [int(x) for x in rng.integers(piece - piece // 8, piece + piece // 8 + 1, 30_000 // piece)]
    col = steps(lens, 3, 40, piece, 25) << np.uint64(shift)
    check(codec, ref, col, tau=0.03)
    check(codec, ref, col, tau=0.1)


def test_very_long_neighbour_after_hulls(codec, ref):
    """A chain of short partitions (hulls built), then a neighbour beyond
    8192 values, then short ones again."""
    rng = np.random.default_rng(7)
    noisy = lambda n: rng.integers(0, 64, n)
    a, b, c = 6000, 9000, 6000
    v = np.concatenate([noisy(a), np.full(b, 32), noisy(c)]) + 9 * np.arange(a + b + c) + 100
    check(codec, ref, v.astype(np.uint32), tau=0.02)


@pytest.mark.parametrize("width", [20, 50])
def test_hulls_that_outgrow(codec, ref, width):
    """Every point of a convex column is a hull vertex: hulls die and unions
    are scanned whole."""
    t = np.arange(12_000, dtype=np.float64)
    rng = np.random.default_rng(width)
    col = (t * t / t[-1] ** 2 * 2.0**width + rng.integers(0, 2, len(t))).astype(np.uint64)
    check(codec, ref, col, tau=0.0)
    check(codec, ref, col, tau=0.02, max_len=5000)


def test_cap_inside_a_batch(codec, ref):
    rng = np.random.default_rng(9)
    col = (np.arange(20_000) * 4 + rng.integers(0, 100, 20_000)).astype(np.uint32)
    for cap in (127, 130, 500, 2049, 2300):
        check(codec, ref, col, tau=0.0, max_len=cap)
