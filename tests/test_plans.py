"""Plans of the batched decode GEMV, on the host: every call is covered once,
and the offsets of its range-checked loads never rely on an offset that the
check does not cover."""
import os
import random
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import plans  # noqa: E402


def shapes(bits):
    rng = random.Random(bits)
    out = [(16, 32, 2), (520, 544, 5), (8208, 6176, 3), (34816, 5120, 16), (5120, 17408, 8), (49200, 6272, 2),
           (65536, 17408, 4), (250, 6144, 16)]
    out += [(rng.randint(1, 70000), 32 * rng.randint(1, 700), rng.randint(1, 16)) for _ in range(40)]
    # the largest matrices of the 32-bit offsets
    if bits == 4:
        out += [(N, K, 2) for N in (16, 31, 16 * 700 + 1) for K in ((1 << 25) - 144, (1 << 25) - 1008, (1 << 24) + 16)]
    else:
        size = 64 * (12 if bits == 3 else 8)
        out += [(16 * (((1 << 31) - 1) // (KC * size)), 128 * KC, 3) for KC in (8, 49, 136, 1000)]
    return out


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_gemv_plan_loads(bits):
    for N, K, B in shapes(bits):
        most = plans.shim().gemv_contract_groups(B, (N + 15) // 16, (K + 127) // 128, 256)
        for m in sorted({1, 2, most}):
            p = plans.gemv_plan(bits, B, N, K, m)
            assert p.ok, (N, K, B)
            T, KC = (N + 15) // 16, (K + 127) // 128
            assert 1 <= p.CPW <= 3 and 1 <= p.KG <= max(1, m) and (p.KG - 1) * p.KCR < KC <= p.KG * p.KCR
            assert p.G == -(-T // p.TPG) * p.KG and 1 <= p.park <= p.TPG
            if p.KCR > p.W * p.CPW:   # passes: every tile of a workgroup is parked
                assert p.park == p.TPG
            for scales in (0, 1):
                assert plans.gemv_bad_loads(bits, B, N, K, m, scales) == 0, (bits, N, K, B, m, scales)


@pytest.mark.parametrize("bits", [2, 3])
def test_gemv_plan_converts_once(bits):
    """LUT, many tiles, more than 48 chunks: no compute unit gets a second
    workgroup (which would convert x again), small batches need no reduction
    launch, and no launch leaves a quarter of the compute units idle."""
    for N in (16384, 49168, 65536, 100000, 147456):
        for K in (6176, 8192, 12288, 17408):
            for B in (2, 3, 4):
                p = plans.gemv_plan(bits, B, N, K)
                assert p.G <= 256 and p.KG == 1, (N, K, B, p)
    for N in (2048, 4096, 5120):
        for K in (12288, 17408):
            assert plans.gemv_plan(bits, 16, N, K).G > 192, (N, K)
