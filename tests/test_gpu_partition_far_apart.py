"""GPU merge scan against the oracle on columns of clusters that lie further
apart than a line spans (2^61).  A batch of unions is sized in one scan of its
values; residuals 2^63 above the smallest value of the batch's later
partitions, on both sides of that, must order as any others do.  Starts are whole numbers: exact."""
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


def clusters(rng, length, slope, noise, centre, low):
    """Noisy lines that begin `noise / 2` below `centre`, each followed by
    some values near `low`."""
    out = []
    for _ in range(24):
        n = int(rng.integers(length // 2, length + 1))
        first = centre - noise // 2
        out += [first + slope * i + int(x) for i, x in enumerate(rng.integers(0, noise, n))]
        out += [low + int(x) for x in rng.integers(0, 4, int(rng.integers(40, 70)))]
    return np.array(out, dtype=np.uint64)


# lines of up to 60 values (every union scanned whole), 400 (hulls) and 3000
@pytest.mark.parametrize("length", [60, 400, 3000])
@pytest.mark.parametrize("slope", [9000, 1 << 40, -(1 << 40)])
@pytest.mark.parametrize("centre,low", [(1 << 63, 0), ((1 << 63) + 1000, 1000), (1 << 62, 0),
                                        ((3 << 62), 1 << 62), ((1 << 64) - (1 << 56), 1 << 59)])
def test_clusters(codec, ref, length, slope, centre, low):
    import torch
    rng = np.random.default_rng(length)
    col = clusters(rng, length, slope, 64, centre, low)
    print(f"[far apart] length={length} slope={slope} centre={centre:#x} low={low:#x}", flush=True)
    for kw in (dict(tau=0.0), dict(tau=0.02)):
        got = codec.partition(torch.from_numpy(col).cuda(), **kw)
        assert np.array_equal(got, ref.partition_greedy(col, **kw))
