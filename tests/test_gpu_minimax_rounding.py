"""GPU parity of the minimax line on nearly straight partitions of ranges
2^50 and up.  There fl(theta) t is off by up to hundreds, so that the stored
line's residuals can be narrower than the exact strip: a search that ended on
the strip's width alone would miss lines that need fewer bits than the
least-squares line.  Bytes equal the oracle's."""
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


def same_blob(codec, ref, col, **kw):
    import torch
    print(f"[minimax rounding] n={len(col)} {kw}", flush=True)
    got = codec.encode(torch.from_numpy(np.ascontiguousarray(col)).cuda(), regressor="minimax",
                       **kw).cpu().numpy()
    assert np.array_equal(got, ref.encode(col, regressor="minimax", **kw))


@pytest.mark.parametrize("values", [
    # least squares needs 9 bits, the minimax line 8; width 261.2 at 645751967822005311 / 5
    (0, 129150393564401187, 258300787128801988, 387451180693203248, 516601574257604195,
     645751967822005313, 774902361386406498, 904052754950807491),
    # 8 and 7 bits; width 135.5
    (0, 283149634046429937, 566299268092859673, 849448902139289680),
])
def test_width_above_the_stored_lines(codec, ref, values):
    same_blob(codec, ref, np.array(values, dtype=np.uint64), fixed_len=len(values))


def lines(rng, length, log2_range, noise_bits):
    """Noisy lines of `length` values of ranges about 2^log2_range, rising
    and falling."""
    out = []
    for bits in noise_bits:
        top = int(rng.integers(1 << (log2_range - 1), 1 << log2_range))
        num, den = top, max(length - 1, 1)
        noise = rng.integers(0, 1 << bits, length)
        v = [num * i // den + int(x) for i, x in zip(range(length), noise)]
        if rng.integers(0, 2):
            v = v[::-1]
        out.append(np.array(v, dtype=np.uint64))
    return out


@pytest.mark.parametrize("log2_range", [50, 51, 52, 53, 54, 56, 57, 58, 59, 60])
@pytest.mark.parametrize("length,count", [(3, 600), (8, 600), (64, 200), (1000, 40), (1025, 12),
                                          (2049, 12), (5000, 12)])
def test_noisy_lines(codec, ref, length, count, log2_range):
    """A few hundred lines of every range and length class: a wavefront with
    16 and 32 values per lane, a workgroup, streamed."""
    rng = np.random.default_rng(100 * length + log2_range)
    noise_bits = [int(b) for b in rng.integers(1, 12, count)]
    same_blob(codec, ref, np.concatenate(lines(rng, length, log2_range, noise_bits)),
              fixed_len=length)
