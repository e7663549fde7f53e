"""GPU merge scan against the oracle where a very long partition merges with
the short ones behind it: smooth curves whose hulls have about 30 to several
hundred vertices, sized from hulls or by scans of the whole.  Starts are whole
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
    print(f"[long head] n={len(col)} {col.dtype} {kw}", flush=True)
    got = codec.partition(torch.from_numpy(np.ascontiguousarray(col)).cuda(), **kw)
    assert np.array_equal(got, ref.partition_greedy(col, **kw))


@pytest.mark.parametrize("n", [60_000, 300_000])
@pytest.mark.parametrize("dtype", [np.uint32, np.uint64])
def test_sorted_normal(codec, ref, n, dtype):
    rng = np.random.default_rng(n)
    col = np.sort(np.clip(np.rint(rng.normal(size=n) * 2.0**26 + 2.0**30), 0, 2**31 - 1)).astype(dtype)
    check(codec, ref, col, tau=0.1)


@pytest.mark.parametrize("rise", [2.0**12, 2.0**16, 2.0**19, 2.0**22, 2.0**44])
@pytest.mark.parametrize("bend", [1, -1])
def test_curve_then_noise(codec, ref, rise, bend):
    """A parabola of 30,000 values (one partition; the higher it rises the
    more of its points are vertices), then noise in short partitions."""
    t = np.arange(30_000, dtype=np.float64)
    head = (t / t[-1]) ** 2 * rise * bend + (rise if bend < 0 else 0) + t
    rng = np.random.default_rng(int(rise) % 1000)
    tail = head[-1] + np.arange(1500) + rng.integers(0, 4, 1500) * max(1.0, rise / 2.0**14)
    col = np.concatenate([head, tail]).astype(np.uint64) + np.uint64(1 << 20)
    for tau in (0.01, 0.03, 0.1):
        check(codec, ref, col, tau=tau)
