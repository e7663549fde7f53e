"""Word offsets and records of encoded columns where the scan over
partitions changes its way: group edges, columns that begin inside a group
and span several, empty columns between them, and enough groups for sums and
prefixes of sums.  Bytes equal the oracle's."""
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


def values(n, seed, dtype=np.uint32):
    rng = np.random.default_rng(seed)
    return (rng.integers(0, 1 << 20, n) >> rng.integers(0, 20, n)).astype(dtype)


@pytest.mark.parametrize("m,L", [(1, 7), (1023, 7), (1024, 5), (1025, 7), (2500, 40),
                                 (32 * 1024, 3), (32 * 1024 + 1, 3), (100_000, 2),
                                 (4096 * 1024, 1), (4096 * 1024 + 1, 1)])
def test_group_edges(codec, ref, m, L):
    import torch
    n = m * L - (L > 1)
    col = values(n, m)
    print(f"[layout] m={m} L={L}", flush=True)
    for regressor in ("minimax", "poly") if m < 100_000 else ("minimax",):
        got = codec.encode(torch.from_numpy(col).cuda(), fixed_len=L, regressor=regressor)
        assert np.array_equal(got.cpu().numpy(), ref.encode(col, fixed_len=L, regressor=regressor))
    if m < 100_000:
        starts = np.concatenate([np.arange(m, dtype=np.uint64) * np.uint64(L), [np.uint64(n)]])
        got = codec.encode(torch.from_numpy(col).cuda(), starts=starts)
        assert np.array_equal(got.cpu().numpy(), ref.encode(col, starts=starts))


@pytest.mark.parametrize("total", [900, 5000, 34_000, 70_000])
def test_columns_across_groups(codec, ref, total):
    import torch
    rng = np.random.default_rng(total)
    sizes, left = [0, 0], total
    while left > 0:
        m = int(min(left, rng.choice([1, 2, 100, 1023, 1024, 1025, 3000, 20000])))
        sizes.append(m)
        left -= m
        if rng.random() < 0.3:
            sizes.append(0)
    sizes.append(0)
    jobs, keep = [], []
    out = torch.zeros(len(sizes), dtype=torch.uint64, device="cuda")
    for i, m in enumerate(sizes):
        L = int(rng.integers(1, 12))
        reg = int(rng.choice([1, 2]))
        col = values(m * L, 31 * i + total, np.uint64)
        d = torch.from_numpy(col).cuda()
        cap = 4096 + 64 * m + 8 * len(col) + 8 * m
        buf = torch.zeros((cap + 15) // 16 * 16, dtype=torch.uint8, device="cuda")
        keep.append((col, d, buf, L, reg))
        jobs.append(P.EncodeJob(d.data_ptr() if m else 0, len(col), 8, 0, L, buf.data_ptr(),
                                buf.numel(), out.data_ptr() + 8 * i, reg, 0))
    print(f"[layout] {len(jobs)} columns, {total} partitions", flush=True)
    codec.check("leco_encode_batch", P.leco_encode_batch(codec.ctx, jobs))
    codec.sync()
    got = out.cpu().numpy()
    for i, (col, d, buf, L, reg) in enumerate(keep):
        want = ref.encode(col, fixed_len=L, regressor=("ls", "minimax", "poly")[reg])
        assert got[i] == len(want)
        assert np.array_equal(buf[: len(want)].cpu().numpy(), want), (i, L, reg, len(col))
