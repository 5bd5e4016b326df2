"""One-pass RMSNorm + quantizer (static scale, K <= 8192): the number of
wavefronts per row follows the number of rows, and must not change a byte."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import dq_layout as L  # noqa: E402
import synth  # noqa: E402
from oracle import norm  # noqa: E402

pytestmark = pytest.mark.gpu

try:
    import paper_2609_26333_amd as dq
except ImportError:  # pragma: no cover
    dq = None


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if dq is None or not torch.cuda.is_available():
        pytest.skip("needs the built HIP library and a GPU")


@pytest.mark.parametrize("K", [16, 512, 528, 1040, 2064, 4096, 5120, 8192])
def test_rmsnorm_rows(K):
    """Rows of a tall input (one wavefront per row) against the same rows alone
    (2, 4 and 8 wavefronts, full and ragged), and eight of them against the
    oracle's codes (a code may differ at a rounding boundary: the oracle's sum
    of squares is exactly rounded)."""
    print("rmsnorm rows", K, flush=True)
    M = 1056
    xb = synth.random_bf16(K, (M, K), outlier_frac=0.005, outlier_factor=30)
    gb = synth.bf16_bits_from_f32((1.0 + 0.2 * synth.random_f32(K + 1, (1, K))).astype(np.float32))[0]
    G = np.float32(0.0125)
    g_d, G_d = torch.from_numpy(gb.view(np.int16)).cuda(), torch.from_numpy(np.array([G], np.float32)).cuda()

    def run(rows):
        x = torch.from_numpy(np.ascontiguousarray(xb[:rows]).view(np.int16)).cuda()
        t = dq.dq_rmsnorm_quantize_act_nvfp4(x, g_d, 1e-5, G_static=G_d)
        q, c, qf, cf = L.nvfp4_unpack(t.codes.cpu().numpy(), t.scales.cpu().numpy(), rows, K)
        assert not qf[rows:].any() and not cf[rows:].any()
        return q, c

    q, c = run(M)
    for rows in (1, 33, 256, 257, 512, 513, 1024, 1025):
        q1, c1 = run(rows)
        assert np.array_equal(q1, q[:rows]) and np.array_equal(c1, c[:rows]), rows
    q_ref, c_ref, _, _ = norm.quantize_rmsnorm_bf16(xb[:8], gb, 1e-5, G)
    assert (q[:8] != q_ref).sum() + (c[:8] != c_ref).sum() <= max(1, 8 * K // 10000)
