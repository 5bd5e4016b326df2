"""LUT GEMV at batch >= 2 (activations in registers), at the edges of its
plan: rows of 1 to 136 chunks (4, 8 and 16 wavefronts, 1 to 3 chunks each,
K groups, passes, wavefronts with one chunk less), one to many row tiles per
workgroup (more than are parked in LDS at once among them), the three batch
widths, both table modes, against the fp64 oracle element by element."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import parity_bounds as PB  # noqa: E402
import plans  # noqa: E402

import synth  # noqa: E402
from oracle import formats, linalg, lut  # noqa: E402

pytestmark = pytest.mark.gpu

try:
    import paper_2609_26333_amd as dq
except ImportError:  # pragma: no cover
    dq = None


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if dq is None or not torch.cuda.is_available():
        pytest.skip("needs the built HIP library and a GPU")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(w, Wq, xb, rows, bits, mode, what):
    """fp32 and bf16 outputs at the given weight rows."""
    B, K = xb.shape
    x = dev(xb.view(np.int16))
    y = dq.dq_decode_gemv(x, Wq, out_kind=dq.OUT_F32)
    yb = dq.dq_decode_gemv(x, Wq, out_kind=dq.OUT_BF16)
    na = dq.dq_decode_gemv_noalloc(x, Wq, out_kind=dq.OUT_F32)
    torch.cuda.synchronize()
    assert torch.equal(y, na) and torch.equal(yb, y.bfloat16())
    if mode == dq.LUT_PER_ROW:
        codes, table = lut.quantize_per_row(w[rows], bits)
        ref, what_hat = linalg.lut_gemv_per_row(xb, codes, table), lut.dequantize_per_row(codes, table)
        bound = PB.gemv_bound(formats.f64_from_bf16_bits(xb), what_hat, K)
    else:
        grid = lut.default_grid(bits)
        if isinstance(w, _Rows):   # the rows' codes under the whole weight's scale
            codes, sb, G = lut.quantize_paper_grid(np.vstack([w[rows], w.largest()]), grid)
            codes, sb = codes[:-1], sb[:-1]
        else:
            codes, sb, G = lut.quantize_paper_grid(w, grid)
            codes, sb = codes[rows], sb[rows]
        ref, what_hat = linalg.lut_gemv_paper(xb, codes, sb, G, grid), lut.dequantize_paper_grid(codes, sb, G, grid)
        bound = PB.gemv_bound(formats.f64_from_bf16_bits(xb), what_hat, K, folded_rel=2.0 ** -11)
    PB.assert_within(y.cpu().numpy()[:, rows], ref, bound, what)


CASES = [(5, 32, 2), (16, 128, 3), (100, 96, 5), (520, 512, 16), (37, 544, 9), (200, 1056, 4), (8208, 1056, 2),
         (8208, 1536, 8), (8200, 1568, 16), (8200, 3072, 7), (8200, 3104, 12), (600, 4096, 2), (9000, 4096, 11),
         (250, 6144, 16), (9000, 6144, 3), (300, 6176, 8), (40, 12288, 16), (2050, 17408, 6), (70, 17408, 2)]


@pytest.mark.parametrize("N,K,B", CASES)
@pytest.mark.parametrize("bits,mode", [(3, 0), (2, 0), (3, 1), (2, 1)])
def test_gemv_batch(N, K, B, bits, mode):
    print("gemv batch", N, K, B, bits, mode, flush=True)
    w = synth.random_f32(N + K, (N, K), 0.02)
    xb = synth.random_bf16(B + K, (B, K), outlier_frac=0.005, outlier_factor=30)
    Wq = dq.dq_pack_lut3(dev(w), bits=bits, mode=mode)
    rows = np.arange(N) if N * K <= 1 << 20 else np.unique(np.r_[0:16, N - 20:N, np.random.default_rng(N).choice(N, 60)])
    check(w, Wq, xb, rows, bits, mode, "gemv batch")


# More tiles per workgroup than are parked at once (9, 18 and 36 at the three
# batch widths), with one K group and with several, and passes over the parked
# tiles (every one of them parked); a ragged last workgroup each.
MANY = [(39900, 3200, 16, "one group"), (79900, 3232, 8, "one group"), (149900, 3200, 3, "one group"),
        (19900, 12000, 16, "groups"), (39900, 12000, 8, "groups"), (149900, 6400, 4, "groups"),
        (49200, 6272, 2, "passes"), (65400, 8224, 4, "passes"), (16200, 6176, 7, "passes"), (100100, 12320, 3, "passes")]


@pytest.mark.parametrize("N,K,B,kind", MANY)
@pytest.mark.parametrize("bits,mode", [(3, 0), (2, 1)])
def test_gemv_batch_many_tiles(N, K, B, kind, bits, mode):
    print("gemv many tiles", N, K, B, kind, bits, mode, flush=True)
    p = plans.gemv_plan(bits, B, N, K, cus=torch.cuda.get_device_properties(0).multi_processor_count)
    assert (p.KG > 1) == (kind == "groups") and (p.KCR > p.W * p.CPW) == (kind == "passes"), p
    assert p.park == p.TPG if kind == "passes" else p.park < p.TPG, p
    g = torch.Generator(device="cuda").manual_seed(3)
    w = torch.randn((N, K), generator=g, device="cuda").mul_(0.02)
    Wq = dq.dq_pack_lut3(w, bits=bits, mode=mode)
    xb = synth.random_bf16(12, (B, K), outlier_frac=0.005, outlier_factor=30)
    T, rng = (N + 15) // 16, np.random.default_rng(5)
    tiles = [0, T - 1, T - 2]   # around the parks and the ends of some workgroups
    for wg in (0, 1, p.G // p.KG - 2, p.G // p.KG - 1):
        tiles += [wg * p.TPG + t for t in (0, p.park - 1, p.park, 2 * p.park, p.TPG - 1) if t < p.TPG]
    tiles = np.unique(np.clip(tiles, 0, T - 1))
    rows = np.unique(np.r_[(tiles[:, None] * 16 + [0, 7, 15]).ravel(), N - 1, rng.choice(N, 40)])
    check(_Rows(w), Wq, xb, rows[rows < N], bits, mode, "gemv many tiles")


class _Rows:
    """Rows of a device tensor by index, on the host."""

    def __init__(self, t):
        self.t = t

    def __getitem__(self, rows):
        return self.t[torch.from_numpy(np.asarray(rows)).cuda()].cpu().numpy()

    def largest(self):
        """The row that holds the largest magnitude."""
        return self.t[self.t.abs().amax(1).argmax()].cpu().numpy()[None]


def test_gemv_batch_scales_per_row():
    """Batch rows of very different magnitudes: each keeps its own scale."""
    N, K, B = 48, 4096, 16
    w = synth.random_f32(1, (N, K), 0.02)
    x = synth.random_f32(2, (B, K)) * np.exp2(np.linspace(-60, 60, B)).astype(np.float32)[:, None]
    xb = synth.bf16_bits_from_f32(x)
    check(w, dq.dq_pack_lut3(dev(w), bits=3), xb, np.arange(N), 3, dq.LUT_PER_ROW, "gemv scales")
