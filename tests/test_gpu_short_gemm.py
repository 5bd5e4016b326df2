"""NVFP4 GEMM on short grids: the kernel that splits K over the wavefronts of
a workgroup, at the edges of its tiles (rows, columns and K steps that end
inside one, wavefronts without a K step, ring cycles that end early) and for
every tile shape, and shapes on the ring kernels' side of the rule, against the
fp64 oracle of the GPU's own operand codes and the oracle quantizer."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import dq_layout as L  # noqa: E402
import parity_bounds as PB  # noqa: E402
import plans  # noqa: E402

import synth  # noqa: E402
from oracle import linalg, nvfp4  # noqa: E402

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


# (M, N, K), and the tile in 32s that a 256-CU device takes for it (None: the
# ring kernels).  Columns that are no multiple of a tile, of 16 or of 4; K from
# a quarter step to 26 steps, so that wavefronts have three steps, one or none.
SHAPES = [((1, 16, 16), None), ((16, 48, 64), None), ((33, 100, 80), None), ((168, 34816, 64), None),
          ((250, 6144, 512), None), ((384, 5120, 640), None), ((160, 8192, 320), None), ((700, 3000, 272), None),
          ((64, 97, 512), (1, 1)), ((65, 224, 528), (1, 1)), ((96, 1000, 1040), (1, 1)), ((130, 352, 2048), (1, 1)),
          ((33, 1000, 272), (1, 1)),
          ((70, 8224, 592), (1, 2)), ((161, 1504, 1616), (1, 2)), ((33, 6200, 1616), (1, 2)),
          ((168, 4096, 576), (2, 2)), ((161, 3040, 528), (2, 2)), ((70, 6200, 592), (2, 2)),
          ((225, 4128, 592), (3, 2)), ((333, 2992, 592), (3, 2)), ((700, 1504, 592), (3, 2)), ((161, 6200, 592), (3, 2)),
          ((100, 8224, 784), (2, 3)), ((500, 2992, 784), (2, 3)), ((300, 4128, 1104), (2, 3)),
          ((333, 4128, 1104), (4, 2)), ((200, 6200, 1040), (4, 2)), ((200, 6176, 1040), (4, 2))]


def test_short_gemm_tiles():
    """Every tile has a shape with ragged rows, and with an NVFP4 and a SwiGLU output."""
    for tile in ((1, 1), (1, 2), (2, 2), (3, 2), (2, 3), (4, 2)):
        mine = [s for s, t in SHAPES if t == tile]
        assert any(N % 16 == 0 and M % 32 for M, N, K in mine) and any(N % 32 == 0 and M % 32 for M, N, K in mine)
        assert any(N % (32 * tile[1]) for M, N, K in mine)


@pytest.mark.parametrize("shape,tile", SHAPES)
def test_short_gemm(shape, tile):
    M, N, K = shape
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus != 256 or plans.gemm_short_tile(M, N, K, cus) == tile
    print("short gemm", M, N, K, flush=True)
    xb = synth.random_bf16(M + N, (M, K), outlier_frac=0.01, outlier_factor=20)
    w = synth.random_f32(N + K, (N, K), 0.02)
    A = dq.dq_quantize_act_nvfp4(dev(xb.view(np.int16)))
    W = dq.dq_pack_nvfp4(dev(w))
    y32 = dq.dq_prefill_gemm(W, A=A, out_kind=dq.OUT_F32)
    yb = dq.dq_prefill_gemm(W, A=A, out_kind=dq.OUT_BF16)
    torch.cuda.synchronize()
    y32, yb = y32.cpu().numpy(), yb.float().cpu().numpy()
    cols = np.arange(N) if N <= 4096 else np.sort(np.random.default_rng(1).choice(N, 700, replace=False))
    qa, ca, Ga = nvfp4.quantize_bf16_activations(xb)
    qw, cw, Gw = nvfp4.quantize_dynamic(w)
    qw, cw = qw[cols], cw[cols]
    ref = linalg.nvfp4_gemm(qa, ca, Ga, qw, cw, Gw)
    bound = PB.fp32_sum_bound(PB.abs_products(nvfp4.dequantize(qa, ca, Ga), nvfp4.dequantize(qw, cw, Gw)), K)
    PB.assert_within(y32[:, cols], ref, bound, "short gemm")
    # bf16: the same sums, rounded to nearest even
    assert np.array_equal(yb, torch.from_numpy(y32).bfloat16().float().numpy())
    G_o = nvfp4.global_scale(0.7 * nvfp4.amax(y32))   # some values saturate
    Gd = dev(np.array([G_o], np.float32))
    if N % 16 == 0:
        Yq = dq.dq_prefill_gemm(W, A=A, out_kind=dq.OUT_NVFP4, G_out_static=Gd)
        torch.cuda.synchronize()
        q, c, qfull, cfull = L.nvfp4_unpack(Yq.codes.cpu().numpy(), Yq.scales.cpu().numpy(), M, N)
        q_ref, c_ref = nvfp4.quantize(y32, G_o)
        assert np.array_equal(c, c_ref) and np.array_equal(q, q_ref)
        assert not qfull[M:].any() and not qfull[:, N:].any() and not cfull[M:].any() and not cfull[:, N // 16:].any()
        assert Yq.G.cpu().numpy()[0] == G_o
    if N % 32 == 0:
        s32 = dq.dq_prefill_gemm(W, A=A, out_kind=dq.OUT_F32, epilogue_flags=dq.EPI_SWIGLU)
        Yq = dq.NvFp4Tensor.empty(M, N // 2)
        Yq.codes.fill_(0xFF)     # the padding has to be written
        Yq.scales.fill_(0xFF)
        dq.dq_prefill_gemm(W, A=A, out_kind=dq.OUT_NVFP4, G_out_static=Gd, epilogue_flags=dq.EPI_SWIGLU, Yq=Yq)
        torch.cuda.synchronize()
        s32 = s32.cpu().numpy()
        blocks = y32.astype(np.float64).reshape(M, N // 32, 2, 16)
        g, u = blocks[:, :, 0], blocks[:, :, 1]
        s_ref = (g / (1.0 + np.exp(-g)) * u).reshape(M, N // 2)
        assert np.all(np.abs(s32 - s_ref) <= 1e-6 * np.abs(s_ref) + 1e-30)   # four fp32 roundings of the same operands
        q, c, qfull, cfull = L.nvfp4_unpack(Yq.codes.cpu().numpy(), Yq.scales.cpu().numpy(), M, N // 2)
        q_ref, c_ref = nvfp4.quantize(s32, G_o)
        assert np.array_equal(c, c_ref) and np.array_equal(q, q_ref)
        assert not qfull[M:].any() and not qfull[:, N // 2:].any()
        assert not cfull[M:].any() and not cfull[:, N // 32:].any()
