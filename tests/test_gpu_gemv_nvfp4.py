"""NVFP4A16 GEMV at the edges of its plan: rows of one scale block to 272 K
steps (odd counts, one to three chunks per wavefront, K groups, passes over the
activations), half row tiles, the three batch widths, both sides of the rule
between the kernels, against the fp64 oracle element by element."""
import ctypes
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import parity_bounds as PB  # noqa: E402
import plans  # noqa: E402

import synth  # noqa: E402
from oracle import formats, linalg, nvfp4  # noqa: E402

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


def check(w, xb, rows):
    """w: on the host, or on the GPU (then only its rows are compared)."""
    (B, K), N = xb.shape, w.shape[0]
    on_gpu = isinstance(w, torch.Tensor)
    Wq = dq.dq_pack_nvfp4(w if on_gpu else dev(w))
    x = dev(xb.view(np.int16))
    y = dq.dq_decode_gemv_nvfp4(x, Wq, out_kind=dq.OUT_F32)
    yb = dq.dq_decode_gemv_nvfp4(x, Wq, out_kind=dq.OUT_BF16)
    yp = torch.empty_like(y)
    d = Wq.desc()
    assert dq.lib().dq_decode_gemv_nvfp4(x.data_ptr(), B, ctypes.byref(d), dq.OUT_F32, yp.data_ptr(), None, 0,
                                         torch.cuda.current_stream().cuda_stream) == dq.DQ_OK
    torch.cuda.synchronize()
    assert torch.equal(y, yp) and torch.equal(yb, y.bfloat16())
    if on_gpu:   # the rows' codes under the whole weight's scale
        G = nvfp4.global_scale(np.float32(w.abs().max().item()))
        q, c = nvfp4.quantize(w[torch.from_numpy(rows).cuda()].cpu().numpy(), G)
    else:
        q, c, G = nvfp4.quantize_dynamic(w)
        q, c = q[rows], c[rows]
    bound = PB.gemv_bound(formats.f64_from_bf16_bits(xb), nvfp4.dequantize(q, c, G), K)
    PB.assert_within(y.cpu().numpy()[:, rows], linalg.nvfp4a16_gemv(xb, q, c, G), bound, "nvfp4 gemv")


CASES = [(5, 16, 2), (16, 48, 16), (33, 64, 5), (100, 80, 3), (47, 144, 9), (520, 512, 16), (40, 1040, 4),
         (4096, 1040, 1), (4112, 1024, 2), (4112, 1040, 2), (4112, 1040, 3), (8192, 1088, 2), (8208, 1104, 2),
         (8200, 1552, 8), (8200, 3088, 7), (8200, 3104, 12), (9000, 4096, 11), (250, 6144, 16), (300, 6160, 3),
         (300, 6160, 1), (2050, 7184, 12), (70, 8208, 2), (40, 12304, 16), (2050, 17408, 6), (70, 17408, 8),
         # both sides of the rule at two, three, four and eight tiles per compute unit, and of the plan's
         # wavefronts per workgroup (4, 8 and 16 for short rows)
         (4112, 528, 1), (8192, 512, 1), (8208, 2064, 1), (8208, 2048, 1), (12304, 784, 2), (12304, 2576, 2),
         (16384, 4112, 3), (5120, 4112, 4), (5120, 4096, 4), (12288, 1040, 2), (16400, 1552, 3), (16400, 784, 8),
         (20496, 2576, 4), (30720, 2064, 2), (32784, 1040, 2), (3072, 4112, 1)]


@pytest.mark.parametrize("N,K,B", CASES)
def test_gemv_nvfp4(N, K, B):
    print("nvfp4 gemv", N, K, B, flush=True)
    w = synth.random_f32(N + K, (N, K), 0.02)
    xb = synth.random_bf16(B + K, (B, K), outlier_frac=0.005, outlier_factor=30)
    rows = np.arange(N) if N * K <= 1 << 20 else np.unique(np.r_[0:33, N - 20:N, np.random.default_rng(N).choice(N, 60)])
    check(w, xb, rows)


# More tiles per workgroup than are parked at once (9, 18 and 36 at the three
# batch widths), with one K group and with several; a ragged last workgroup each
MANY = [(39900, 3216, 16, 1), (79900, 3200, 7, 1), (149900, 3200, 1, 1), (19900, 12016, 16, 2), (39900, 8208, 6, 2),
        (149900, 6416, 2, 2)]


@pytest.mark.parametrize("N,K,B,groups", MANY)
def test_gemv_nvfp4_many_tiles(N, K, B, groups):
    print("nvfp4 gemv many tiles", N, K, B, flush=True)
    T = (N + 15) // 16
    need = dq.dq_decode_gemv_nvfp4_workspace_size(B, dq.NvFp4Tensor.empty(N, K))
    p = plans.gemv_plan(4, B, N, K, most=max(1, need // (T * B * 64)),
                        cus=torch.cuda.get_device_properties(0).multi_processor_count)
    assert p.KG == groups and p.park < p.TPG and p.KCR <= p.W * p.CPW, p
    g = torch.Generator(device="cuda").manual_seed(3)
    w = torch.randn((N, K), generator=g, device="cuda").mul_(0.02)
    xb = synth.random_bf16(12, (B, K), outlier_frac=0.005, outlier_factor=30)
    tiles = [0, T - 1, T - 2]
    for wg in (0, 1, p.G // p.KG - 2, p.G // p.KG - 1):
        tiles += [wg * p.TPG + t for t in (0, p.park - 1, p.park, 2 * p.park, p.TPG - 1) if t < p.TPG]
    tiles = np.unique(np.clip(tiles, 0, T - 1))
    rows = np.unique(np.r_[(tiles[:, None] * 16 + [0, 7, 15]).ravel(), N - 1, np.random.default_rng(5).choice(N, 40)])
    check(w, xb, rows[rows < N])


@pytest.mark.parametrize("N,B", [(3, 2), (2, 11), (2, 12), (1, 16)])
def test_gemv_nvfp4_widest_rows(N, B):
    """Rows past the batched kernel's offsets (2^25 columns): the K-group kernel,
    two widths of the group.  x is zero but for a few scale blocks (the first,
    the last, both sides of group edges and of 2^24), the weights are not."""
    print("nvfp4 gemv widest rows", N, B, flush=True)
    K = (1 << 25) + 16
    assert not plans.gemv_plan(4, B, N, K, most=1).ok
    at = [0, 1008, 1024, 2032, 2048, (1 << 24) - 16, 1 << 24, (1 << 25) - 16, 1 << 25]
    cols = np.concatenate([np.arange(k, k + 16) for k in at])
    on = torch.from_numpy(cols).cuda()
    g = torch.Generator(device="cuda").manual_seed(N)
    w = torch.randn((N, K), generator=g, device="cuda").mul_(0.02)
    xb = synth.random_bf16(B, (B, len(cols)), outlier_frac=0.02, outlier_factor=30)
    x = torch.zeros((B, K), dtype=torch.int16, device="cuda")
    x[:, on] = dev(xb.view(np.int16))
    Wq = dq.dq_pack_nvfp4(w)
    y = dq.dq_decode_gemv_nvfp4(x, Wq, out_kind=dq.OUT_F32)
    yb = dq.dq_decode_gemv_nvfp4(x, Wq, out_kind=dq.OUT_BF16)
    torch.cuda.synchronize()
    assert torch.equal(yb, y.bfloat16())
    G = nvfp4.global_scale(np.float32(w.abs().max().item()))
    q, c = nvfp4.quantize(w[:, on].cpu().numpy(), G)
    bound = PB.gemv_bound(formats.f64_from_bf16_bits(xb), nvfp4.dequantize(q, c, G), len(cols))
    PB.assert_within(y.cpu().numpy(), linalg.nvfp4a16_gemv(xb, q, c, G), bound, "nvfp4 gemv, widest rows")


def test_gemv_nvfp4_scales_per_row():
    """Batch rows of very different magnitudes: each keeps its own scale."""
    N, K, B = 48, 4096, 16
    x = synth.random_f32(2, (B, K)) * np.exp2(np.linspace(-60, 60, B)).astype(np.float32)[:, None]
    check(synth.random_f32(1, (N, K), 0.02), synth.bf16_bits_from_f32(x), np.arange(N))


@pytest.mark.parametrize("out_kind,dtype", [(dq.OUT_F32, torch.float32), (dq.OUT_BF16, torch.bfloat16)] if dq else [])
@pytest.mark.parametrize("N,B", [(5, 3), (1, 1), (300, 7)])
def test_gemv_nvfp4_no_columns(N, B, out_kind, dtype):
    """K = 0: zeros in y and nothing behind it (odd element counts)."""
    Wq = dq.NvFp4Tensor.empty(N, 0)
    x = torch.empty((B, 0), dtype=torch.bfloat16, device="cuda")
    buf = torch.full((B * N + 8,), 7.0, dtype=dtype, device="cuda")
    dq.dq_decode_gemv_nvfp4(x, Wq, out_kind=out_kind, y=buf[:B * N].view(B, N))
    torch.cuda.synchronize()
    assert not buf[:B * N].any() and (buf[B * N:] == 7.0).all()
