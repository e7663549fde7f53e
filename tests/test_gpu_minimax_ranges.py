"""GPU parity of the minimax search where it changes its arithmetic or its
kernel: ranges either side of the binary64 limit of each partition size
(2^32 up to 1024 values, 2^30 up to 2048, 2^28 up to 4096, 2^24 up to 16384),
partition lengths either side of each kernel's largest, point sets that take
the search the most steps, and edges whose fractions round differently
(differences beyond 2^53).  Bytes equal the oracle's."""
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


def same_blob(codec, ref, col, L):
    import torch
    print(f"[minimax ranges] n={len(col)} {col.dtype} L={L}", flush=True)
    got = codec.encode(torch.from_numpy(np.ascontiguousarray(col)).cuda(), fixed_len=L,
                       regressor="minimax").cpu().numpy()
    assert np.array_equal(got, ref.encode(col, fixed_len=L, regressor="minimax"))


@pytest.mark.parametrize("L,log2_range", [(1024, 32), (1000, 32), (2048, 30), (1025, 30),
                                          (4096, 28), (2049, 28), (4097, 24), (10_000, 24)])
@pytest.mark.parametrize("over", [-1, 0])
def test_binary64_limit(codec, ref, L, log2_range, over):
    """Every partition's range is exactly 2^log2_range + over: noise on a
    bend, its ends and middle pinned to the range's ends."""
    rng = np.random.default_rng(1000 * L + log2_range + over)
    top = (1 << log2_range) + over
    part = 3
    t = np.arange(L)
    cols = []
    for _ in range(part):
        v = (np.abs(t - L / 2) / L * top).astype(np.int64) + rng.integers(0, top // 3, L)
        v = np.clip(v, 0, top)
        v[rng.integers(0, L)] = 0
        v[(int(np.argmin(v)) + 1 + rng.integers(0, L - 1)) % L] = top
        assert v.max() - v.min() == top
        cols.append(v)
    col = np.concatenate(cols + [cols[0][: L // 3 + 1]]).astype(np.uint64) + np.uint64(1 << 45)
    same_blob(codec, ref, col, L)
    if top < 1 << 32:
        same_blob(codec, ref, (col - col.min()).astype(np.uint32), L)


@pytest.mark.parametrize("L", [2, 3, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097])
def test_lengths(codec, ref, L):
    rng = np.random.default_rng(L)
    n = 3 * L + L // 2 + 1
    col = (np.arange(n) * 5 + rng.integers(0, 200, n)).astype(np.uint32)
    same_blob(codec, ref, col, L)
    same_blob(codec, ref, col.astype(np.uint64) << np.uint64(25), L)


@pytest.mark.parametrize("L", [64, 1024, 2000, 4096])
@pytest.mark.parametrize("bits", [22, 45])
def test_facing_curves(codec, ref, L, bits):
    """Even points on a concave curve above, odd ones on a convex one below:
    every slope between is a bend (about 16 steps)."""
    x = np.arange(L, dtype=np.float64)
    top = 2.0 ** bits
    ups = [np.sqrt(np.maximum(0.0, 1 - ((x - L * 0.3) / L) ** 2)), -(2.0 ** (x * 20.0 / L)) / 2.0**20,
           np.log(x + 1) / 10, -1.0 / (x + 1)]
    downs = [2.0 ** (x * 20.0 / L) / 2.0**20, (x / L) ** 6, 1.0 / (x + 1)]
    col = np.concatenate([np.where(x % 2 == 0, u * top + 3 * top, d * top + top / 2)
                          for u in ups for d in downs]).astype(np.uint64)
    same_blob(codec, ref, col, L)


def test_fractions_beyond_2_53(codec, ref):
    """Parallel upper and lower edges and collinear runs with differences
    above 2^53, where fl(dy) / fl(dt) depends on which points span the edge."""
    rng = np.random.default_rng(53)
    for L in (5, 6, 9, 300):
        cols = []
        for _ in range(40):
            s = int(rng.integers(1 << 53, 1 << 56)) * 2 + 1 if L < 20 else int(rng.integers(1 << 50, 1 << 51)) * 2 + 1
            h = int(rng.integers(1 << 54, 1 << 56))
            t = [int(i) for i in range(L)]
            v = [i * s + (h if i % 3 == 0 else 0 if i % 3 == 1 else int(rng.integers(0, h))) for i in t]
            if rng.integers(0, 2):
                v = [max(v) - y for y in v]
            cols.append(np.array(v, dtype=np.uint64) + np.uint64(1 << 62))
        same_blob(codec, ref, np.concatenate(cols), L)
