"""One-pass encoders that count late partitions themselves, where the column
is not a single one of fixed lengths: tables of columns of both types (the
look-back ends at each column's first partition), empty columns between,
constants forced, and variable starts.  With no reads allowed nearly every
partition counts its predecessors.  Bytes equal the oracle's."""
from __future__ import annotations

import os

import numpy as np
import pytest

import paper_2306_15374_amd as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=["0", "256"])
def codec(request):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    keys = {"LECO_ENCODE_FUSED": "1", "LECO_ENCODE_FUSED_WAVE": "1", "LECO_LOOKBACK_POLLS": request.param}
    old = {k: os.environ.get(k) for k in keys}
    os.environ.update(keys)  # read when the context is created
    try:
        c = P.Codec(0)
    finally:
        for k, v in old.items():
            if v is None:
                del os.environ[k]
            else:
                os.environ[k] = v
    yield c
    c.close()


def column(rng, n, dtype):
    col = np.cumsum(rng.integers(0, 1 << int(rng.integers(1, 14)), n)).astype(np.uint64)
    return col.astype(np.uint32) if dtype == 4 else col + np.uint64(int(rng.integers(0, 1 << 60)))


# partitions of a wavefront each, and of a workgroup each (registers half and all full)
@pytest.mark.parametrize("L", [33, 1024, 2049, 4096])
def test_table(codec, ref, L):
    import torch
    rng = np.random.default_rng(L)
    spec = []  # values, width, constant forced
    for i in range(40):
        n = int(rng.choice([0, 1, L - 1, L, L + 1, 7 * L + 3, 70 * L + 5]))
        spec.append((n, int(rng.choice([4, 8])), int(rng.integers(0, 4) == 0)))
    cols = [column(rng, n, w) for n, w, _ in spec]
    dev = [torch.from_numpy(c).cuda() if len(c) else None for c in cols]
    sizes = torch.zeros(len(spec), dtype=torch.int64, device="cuda")
    blobs, jobs = [], []
    for i, (n, w, const) in enumerate(spec):
        part, _ = P.make_partitioning(L, force_constant=bool(const))
        blobs.append(torch.zeros(P.leco_max_blob_bytes(n, w, part), dtype=torch.uint8, device="cuda"))
        jobs.append(P.EncodeJob(dev[i].data_ptr() if n else None, n, w, const, L, blobs[i].data_ptr(),
                                blobs[i].numel(), sizes.data_ptr() + 8 * i, 0, 0))
    print(f"[look-back tables] L={L} values={[s[0] for s in spec]}", flush=True)
    for _ in range(3):
        codec.check("leco_encode_batch", P.leco_encode_batch(codec.ctx, jobs))
        codec.sync()
        for c, (n, w, const), b, size in zip(cols, spec, blobs, sizes.cpu().tolist()):
            assert np.array_equal(b[:size].cpu().numpy(), ref.encode(c, fixed_len=L, force_constant=bool(const)))
            b.zero_()


@pytest.mark.parametrize("longest", [40, 1024, 4096])
@pytest.mark.parametrize("dtype", [4, 8])
@pytest.mark.parametrize("const", [False, True])
def test_variable_starts(codec, ref, longest, dtype, const):
    import torch
    rng = np.random.default_rng(longest + dtype)
    lens = rng.integers(1, longest + 1, 300)
    lens[7] = longest
    starts = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    col = column(rng, int(starts[-1]), dtype)
    print(f"[look-back tables] variable, longest {longest}, width {dtype}, const {const}", flush=True)
    for _ in range(3):
        got = codec.encode(torch.from_numpy(col).cuda(), starts=starts, force_constant=const)
        assert np.array_equal(got.cpu().numpy(), ref.encode(col, starts=starts, force_constant=const))
