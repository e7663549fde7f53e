"""GPU parity of the polynomial encode's workgroup fit above its narrow range,
where the line is fitted with the range already known: ranges either side of
the next limits (2^30 the narrow sums, 2^50 the polynomials, 2^61 the line),
partitions of one to three values and of more than 4096 in the same launch,
and forced constants.  Bytes equal the oracle's."""
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
    print(f"[poly wide] n={len(col)} {col.dtype}", flush=True)
    got = codec.encode(torch.from_numpy(np.ascontiguousarray(col)).cuda(), regressor="poly", **kw)
    assert np.array_equal(got.cpu().numpy(), ref.encode(col, regressor="poly", **kw))


def part(rng, length, top):
    """A cubic, a line or noise of range exactly `top` (one value: 0)."""
    t = np.arange(length, dtype=object)
    kind, d = int(rng.integers(0, 3)), max(length - 1, 1)
    if kind == 0:
        v = [int(x) ** 3 * top // d**3 for x in t]
    elif kind == 1:
        v = [int(x) * top // d for x in t]
    else:
        v = [int(x) % (top + 1) for x in rng.integers(0, 1 << 63, length, dtype=np.uint64)]
    noise = rng.integers(0, 8, length)
    v = [min(x + int(e), top) for x, e in zip(v, noise)]
    v[0], v[-1] = 0, top if length > 1 else 0
    return v[:: 1 if rng.integers(0, 2) else -1]


@pytest.mark.parametrize("top", [(1 << 28) - 1, 1 << 28, (1 << 30) - 1, 1 << 30, (1 << 32) - 1, (1 << 50) - 1,
                                 1 << 50, (1 << 61) - 1, 1 << 61, (1 << 64) - 1])
def test_limits(codec, ref, top):
    rng = np.random.default_rng(top % (1 << 31))
    for L in (2049, 4095, 4096):
        col = np.array(sum((part(rng, L, top) for _ in range(6)), part(rng, L // 2, top)), dtype=np.uint64)
        check(codec, ref, col, fixed_len=L)
        if top < 1 << 32:
            check(codec, ref, col.astype(np.uint32), fixed_len=L)
    lens = [1, 2, 3, 4, 4096, 5000, 1, 2, 3, 700, 4097, 2, 1]
    col = np.array(sum((part(rng, n, top) for n in lens), []), dtype=np.uint64)
    starts = np.cumsum([0] + lens).astype(np.uint64)
    check(codec, ref, col, starts=starts)
    check(codec, ref, col, starts=starts, force_constant=True)
