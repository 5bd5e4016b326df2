// The kernels' plans (plain C++ headers of csrc/) behind a C interface, for
// tests/plans.py.
#include <cstdint>

#include "gemm_plan.hpp"
#include "gemv_plan.hpp"

extern "C" {

int64_t gemv_contract_groups(int64_t B, int64_t T, int64_t KC, int64_t cus) {
  return dq::contract_groups(B, T, KC, cus);
}

// out: ok, BV, W, CPW, KG, KCR, TPG, G, park
void gemv_plan(int bits, int64_t B, int64_t T, int64_t KC, int64_t most, int64_t cus, int64_t* out) {
  const dq::BatchedPlan p = dq::plan_batched(bits, B, T, KC, most, cus);
  const int64_t v[9] = {p.ok, p.BV, p.W, p.CPW, p.KG, p.KCR, p.TPG, p.G, p.park};
  for (int i = 0; i < 9; ++i) out[i] = v[i];
}

// Walks the code (scales = 0) or block-scale loads of the first and the last
// workgroups of a call as the batched kernel issues them and counts those whose
// offsets the range check of a raw buffer load does not cover: a uniform offset
// past the buffer, a sum of 2^32 or more, a wanted load that does not lie
// inside, an unwanted one that does.  Returns the count.
int64_t gemv_bad_loads(int bits, int64_t B, int64_t T, int64_t KC, int64_t KT, int64_t most, int64_t cus, int scales) {
  const dq::BatchedPlan p = dq::plan_batched(bits, B, T, KC, most, cus);
  if (!p.ok) return -1;
  const int chunk_bytes = scales ? 128 : 64 * (bits == 3 ? 12 : 8), tile_bytes = scales ? 128 : 1024;
  // the largest lane offset and size of a load
  const int32_t lane = bits == 4 ? (scales ? 60 : 32 * 15 + 8 * 3) : scales ? 124 : 63 * (bits == 3 ? 12 : 8);
  const int32_t size = bits == 4 ? (scales ? 4 : 8) : scales ? 4 : bits == 3 ? 12 : 8;
  int64_t bad = 0;
  for (int64_t b = 0; b < p.G; ++b) {
    if (b >= 4 * p.KG && b < p.G - 4 * p.KG) continue;
    const int kg = (int)(b % p.KG), tg = (int)(b / p.KG);
    const int t0 = (int)(tg * p.TPG), nt = (int)std::min<int64_t>(p.TPG, T - t0);
    const int c0 = (int)(kg * p.KCR), nc = (int)std::min<int64_t>(p.KCR, KC - c0);
    const int p0 = t0 >> 1, np = ((t0 + nt + 1) >> 1) - p0;
    const int64_t records = bits == 4 ? (int64_t)np * KT * tile_bytes : T * KC * chunk_bytes;
    if (records >= ((int64_t)1 << 32)) ++bad;
    for (int cp = c0; cp < c0 + nc; cp += (int)(p.W * p.CPW))
      for (int wave = 0; wave < p.W; ++wave) {
        const int nu = std::min<int>((int)p.CPW, (int)((c0 + nc - cp - wave + p.W - 1) / p.W));
        for (int t = 0; t < nt + dq::kAhead; ++t) {
          if (t >= 4 && t < nt - 4) continue;
          for (int u = 0; u < p.CPW; ++u) {
            const bool ok = t < nt && u < nu;
            const int c = cp + u * (int)p.W + wave;
            for (int h = 0; h < (bits == 4 ? 2 : 1); ++h) {
              const bool want = bits == 4 ? ok && 2 * c + h < KT : ok;
              dq::LoadAt a;
              if (bits == 4) {
                const int pair = ((t0 + t) >> 1) - p0, half = (t0 + t) & 1;
                a = dq::nvfp4_step_at(ok, dq::nvfp4_chunk_at(ok, pair, (int)KT, c, half), 2 * c + h, (int)KT, h, lane, lane);
                if (scales) a = dq::LoadAt{a.lane_scale, a.uniform / 8, 0};
              } else {
                a = dq::lut_chunk_at(want, t0 + t, (int)KC, c, lane, lane);
                a = dq::LoadAt{scales ? a.lane_scale : a.lane, a.uniform * chunk_bytes, 0};
              }
              const int64_t l = (uint32_t)a.lane, s = (uint32_t)a.uniform;
              if (s > records || l + s >= ((int64_t)1 << 32)) ++bad;
              else if (want ? l + s + size > records : l < records - s) ++bad;
            }
          }
        }
      }
  }
  return bad;
}

// rows * 100 + columns of the short-grid tile in 32s, or -1 for the ring kernels
int gemm_short_tile(int64_t M, int64_t N, int64_t K, int64_t cus) {
  const int f = dq::choose_short(M, N, K, cus);
  return f < 0 ? -1 : dq::kShortFits[f].tm * 100 + dq::kShortFits[f].tn;
}

}  // extern "C"
