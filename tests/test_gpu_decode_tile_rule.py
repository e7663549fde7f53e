"""Column sizes and ranges on both sides of the rule that shrinks the decode
tile until every CU has three workgroups, and that grows it from 256 values
where a launch has very many.  Decoded values are whole numbers: exact."""
from __future__ import annotations

import numpy as np
import pytest

import paper_2306_15374_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,L,regressor", [
    (2047, 1000, "ls"),
    (2049, 1, "ls"),
    (768 * 2048 + 1, 4096, "ls"),
    (768 * 4096 - 1, 128, "ls"),
    (2048 * 256 + 5, 1, "ls"),
    (2048 * 512 + 7, 2, "ls"),
    (768 * 2048 - 3, 1000, "poly"),
])
def test_decode_at_rule_edges(n, L, regressor):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n)
    col = (3 * np.arange(n) + rng.integers(0, 1 << 16, n)).astype(np.uint32)
    print(f"[tile rule] n={n} L={L}", flush=True)
    codec = P.Codec(0)
    try:
        blob = codec.encode(torch.from_numpy(col).cuda(), fixed_len=L, regressor=regressor)
        assert np.array_equal(codec.decode_all(blob).cpu().numpy(), col)
        for b, e in ((0, n), (0, 1), (n - 1, n), (n // 3, n // 3 + n // 2), (1, min(n, 2050))):
            assert np.array_equal(codec.decode_range(blob, b, e).cpu().numpy(), col[b:e])
    finally:
        codec.close()
