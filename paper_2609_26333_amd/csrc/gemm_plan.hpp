// Choice between the ring kernels and the short-grid kernel of the NVFP4 GEMM
// (gemm.hip), and of the short grid's tile.  Plain C++, so that the CPU tests
// compile it too.
#pragma once

#include <cstdint>

namespace dq {

inline int64_t short_tiles(int64_t n, int t) { return (n + 32 * t - 1) / (32 * t); }

// Modelled time (us) of a grid, for the choice between the kernels.  Both
// sides were measured on 230 combinations of M = 16 .. 4096 with the 8B and
// 27B linears and 1024 x 4096, 1024 x 16384, 3072 x 768; the model is within
// 7-10 % of either, and the choice within 1 % of the faster kernel on average
// (on 460 random shapes up to 8192 rows, within 1.8 % of the fastest of all).
// Ring kernels: per K step, by resident workgroups (1 or 2 per compute unit)
// and then by the total of 256 x 128 tiles.
inline double ring_time(int64_t M, int64_t N, int64_t KT, int64_t cus) {
  const int64_t t = ((M + 255) / 256) * ((N + 127) / 128);
  if (t <= cus) {
    const int64_t half = ((M + 127) / 128) * ((N + 127) / 128);   // 128 x 128 tiles
    return 3.0 + (half <= cus ? 0.50 : 0.90) * (double)KT;
  }
  const double x = (double)t * 256.0 / (double)cus;
  return 3.0 + (t <= 2 * cus ? 1.1 + 0.0008 * x : 0.55 + 0.0026 * x) * (double)KT;
}

// Short-grid tiles: `conc` workgroups per compute unit (by registers); `fixed`
// per round of them (ring fill, reduction, store), `step` per K step and
// workgroup on the fullest compute unit, growing by `crowd` with their number.
struct ShortFit {
  int tm, tn, conc;
  double fixed, step, crowd;
};

constexpr int kNumShortFits = 6;
constexpr ShortFit kShortFits[kNumShortFits] = {{1, 1, 2, 1.65, 0.0439, 0.0},  {1, 2, 2, 2.26, 0.0626, 0.06},
                                                {2, 2, 1, 2.55, 0.0895, 0.33}, {3, 2, 2, 3.19, 0.1286, 0.14},
                                                {2, 3, 2, 3.68, 0.1279, 0.16}, {4, 2, 1, 4.53, 0.1454, 0.40}};

inline double short_time(const ShortFit& f, int64_t M, int64_t cols, int64_t KT, int64_t cus) {
  const int64_t tiles = short_tiles(M, f.tm) * short_tiles(cols, f.tn);
  const double rounds = (double)((tiles + cus * f.conc - 1) / (cus * f.conc)), load = (double)((tiles + cus - 1) / cus);
  return 3.0 + f.fixed * rounds + f.step * (double)KT * load * (1.0 + f.crowd * (1.0 - 1.0 / load));
}

// The short-grid tile to use (an index of kShortFits), or -1 for the ring
// kernels: the faster of the two by the models, 5 % to the ring kernels.
// Measured, bf16 out, M = 168: 27B o 42.1 -> 13.3 us, q/k/v 42.6 -> 17.4, down
// 130 -> 37.3, gate/up 109 -> 67; 8B up 38 -> 23; at M = 1024 down 222 -> 162,
// o 70 -> 55 and gate/up 294 against 313 with the short grid (not used).
// (Columns in whole 128s: the same tile, and so the same sums, whatever the
// output kind.  The tile, and with it the split of K, follows M: a row's last
// bits depend on how many rows come with it.)
inline int choose_short(int64_t M, int64_t N, int64_t K, int64_t cus) {
  const int64_t KT = (K + 63) / 64, cols = (N + 127) / 128 * 128;
  if (KT == 0) return -1;
  double best = 0.95 * ring_time(M, N, KT, cus);
  int pick = -1;
  for (int f = 0; f < kNumShortFits; ++f) {
    const double t = short_time(kShortFits[f], M, cols, KT, cus);
    if (t < best) {
      best = t;
      pick = f;
    }
  }
  return pick;
}

}  // namespace dq
