"""Per-row LUT packing at the edges of its selection: rows whose bin
boundaries fall on ties, whose values crowd one histogram bucket (narrowed by
finer histograms) or spread over the whole fp32 range, and row lengths at the
ends of every kernel's range.  Codes and entries equal the oracle's, bit for bit."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import dq_layout as L  # noqa: E402

from oracle import lut  # noqa: E402

pytestmark = pytest.mark.gpu

try:
    import paper_2609_26333_amd as dq
except ImportError:  # pragma: no cover
    dq = None


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if dq is None or not torch.cuda.is_available():
        pytest.skip("needs the built HIP library and a GPU")


def rows(K):
    """One row of each kind (finite, and with entries inside fp16's range)."""
    rng = np.random.default_rng([7, K])
    z = rng.standard_normal(K, dtype=np.float32)
    out = [0.02 * z,                                             # Gaussian
           np.zeros(K), np.full(K, -1.5),                        # constant
           np.where(np.arange(K) % 3 == 0, 0.25, -0.75),         # two values, uneven
           np.round(2.0 * z) / 2.0,                              # a few values, ties on every boundary
           np.sort(z), -np.sort(z),                              # ordered
           np.where(np.arange(K) == K // 2, 30000.0, z),         # one outlier: the buckets widen
           np.where(np.arange(K) % 16 == 0, 3000.0 * z, 1e-3 * z),   # a wide tail over a crowded middle
           z * np.float32(1e-40), z * np.float32(1e-30),         # fp32 subnormals; far below fp16
           np.exp(8.0 * z.clip(-8, 1.2)) * np.sign(rng.standard_normal(K)),   # many octaves
           np.where(z > 0, np.float32(0.0), np.float32(-0.0)),   # zeros of both signs
           np.where(np.abs(z) < 0.7, 0.0, z)]                    # half zeros
    return np.stack(out).astype(np.float32)


# the ends of each kernel's row lengths (1024, 2048, 4096, 5120 | 6144, 8192,
# 12288 | 16384, 20480, 32768) and lengths that are not a multiple of a
# 128-column chunk
@pytest.mark.parametrize("K", [32, 96, 1024, 1056, 2048, 4064, 4096, 4128, 5120, 5152, 6144, 8224, 12288, 12320, 17408,
                               20480, 32768])
@pytest.mark.parametrize("bits", [3, 2])
def test_pack_lut_rows(K, bits):
    print("pack rows", K, bits, flush=True)
    w = rows(K)
    N = w.shape[0]
    codes, table = lut.quantize_per_row(w, bits)
    Wq = dq.dq_pack_lut3(torch.from_numpy(w).cuda(), bits=bits, mode=dq.LUT_PER_ROW)
    torch.cuda.synchronize()
    entries = Wq.lut.cpu().numpy().view(np.uint16).reshape(-1, 1 << bits)
    assert np.array_equal(entries[:N], table.view(np.uint16))
    assert not entries[N:].any()
    raw = Wq.codes.cpu().numpy()
    # the padding rows and columns hold code 0
    full = L.lut_codes_unpack(raw, (N + 15) // 16 * 16, (K + 127) // 128 * 128, bits)
    assert np.array_equal(full[:N, :K], codes)
    assert not full[N:].any() and not full[:, K:].any()


def crowded_rows(K):
    """Rows whose thresholds share crowded buckets, part after some of the
    rounds that narrow them, and end on keys one apart, equal, or far apart."""
    rng = np.random.default_rng([13, K])
    z = rng.standard_normal(K, dtype=np.float32)
    far = np.arange(K) == K - 1   # widens the buckets: the others fall into one or two

    def ulps(start, n):   # n neighbouring floats, over and over
        return (np.float32(start).view(np.int32) + rng.integers(0, n, K).astype(np.int32)).view(np.float32)

    out = [np.where(far, 50.0 * K, z),                           # both signs, each in one bucket
           np.where(far, -50.0 * K, np.abs(z)),                  # the positive one alone
           np.where(far, 50.0 * K, ulps(1.0, 7)), np.where(far, 50.0 * K, ulps(-1.0, 200)),   # keys one apart
           np.where(far, 50.0 * K, ulps(1.0, 128 * 128)), np.where(far, 50.0 * K, ulps(0.9, 128 * 128 + 1)),
           np.where(far, 50.0 * K, np.where(z > 0, ulps(3.0, 3), ulps(-1e-20, 1000))),   # two far clusters
           np.where(far, 50.0 * K, np.where(z > 0.3, 1.0, z)),   # a tie beside single keys
           np.exp2(rng.uniform(-140.0, 14.0, K)) * np.sign(z),   # every octave, both signs
           np.where(far, 50.0 * K, np.exp2(rng.uniform(-140.0, 3.0, K)))]
    return np.stack(out).astype(np.float32)


@pytest.mark.parametrize("K", [1024, 2048, 4096, 5120, 8192, 12288, 16896, 20480, 32768])   # one per kernel
@pytest.mark.parametrize("bits", [3, 2])
def test_pack_lut_rows_crowded(K, bits):
    print("pack crowded rows", K, bits, flush=True)
    w = crowded_rows(K)
    codes, table = lut.quantize_per_row(w, bits)
    assert np.isfinite(table).all()
    Wq = dq.dq_pack_lut3(torch.from_numpy(w).cuda(), bits=bits, mode=dq.LUT_PER_ROW)
    torch.cuda.synchronize()
    assert np.array_equal(Wq.lut.cpu().numpy().view(np.uint16).reshape(-1, 1 << bits)[:len(w)], table.view(np.uint16))
    assert np.array_equal(L.lut_codes_unpack(Wq.codes.cpu().numpy(), len(w), K, bits), codes)


def test_pack_lut_rows_many_tiles():
    """More row tiles than one group of eight, and a ragged last one."""
    rng = np.random.default_rng(11)
    w = (0.02 * rng.standard_normal((9 * 16 + 5, 160))).astype(np.float32)
    codes, table = lut.quantize_per_row(w, 3)
    Wq = dq.dq_pack_lut3(torch.from_numpy(w).cuda(), bits=3, mode=dq.LUT_PER_ROW)
    torch.cuda.synchronize()
    assert np.array_equal(L.lut_codes_unpack(Wq.codes.cpu().numpy(), w.shape[0], w.shape[1], 3), codes)
    assert np.array_equal(Wq.lut.cpu().numpy().view(np.uint16).reshape(-1, 8)[:w.shape[0]], table.view(np.uint16))
