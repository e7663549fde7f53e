"""GPU merge scan against the oracle where chains of merges end early: the
values that a batch takes follow the lengths of the last merged partitions,
and only unions that a line is fitted to are scanned.  Short and long chains
in turn, near each other and further apart than a line spans.  Starts are
whole numbers: exact."""
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


@pytest.mark.parametrize("lens", [(3,), (5, 8), (31, 32, 33), (40,), (63, 65), (4, 300), (4, 4, 300, 20),
                                  (127, 129), (256, 10), (6, 1500)])
@pytest.mark.parametrize("spread", [12, 30, 62, 64])
def test_chains(codec, ref, lens, spread):
    import torch
    rng = np.random.default_rng(1000 * spread + len(lens) + lens[0])
    col = []
    while len(col) < 12_000:
        for n in lens:
            level = int(rng.integers(0, 1 << 32)) << 32 | int(rng.integers(0, 1 << 32))
            level >>= 64 - spread
            slope = int(rng.integers(0, 9))
            col += [(level + slope * i + int(x)) % (1 << 64) for i, x in enumerate(rng.integers(0, 32, n))]
    col = np.array(col, dtype=np.uint64)
    d = torch.from_numpy(col).cuda()
    for kw in (dict(tau=0.0), dict(tau=0.04), dict(tau=0.1, start_positions=True),
               dict(tau=0.02, max_len=200)):
        print(f"[chains] lens={lens} spread={spread} {kw}", flush=True)
        assert np.array_equal(codec.partition(d, **kw), ref.partition_greedy(col, **kw))
