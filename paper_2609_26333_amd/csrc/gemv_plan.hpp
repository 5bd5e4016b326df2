// Plan of the batched decode GEMV (gemv.hip): how a call is split over K groups,
// workgroups and wavefronts, and the offsets of the kernel's range-checked
// loads.  Plain C++ apart from the function attributes, so that the CPU tests
// compile it too.
#pragma once

#include <algorithm>
#include <cstdint>

#ifdef __HIP__
#define DQ_HOST_DEVICE __host__ __device__
#else
#define DQ_HOST_DEVICE
#endif

namespace dq {

struct BatchPlan {
  int KG, KCR, TPG;   // K groups, chunks per K group, tiles per workgroup
  int tiles, KC;
  int KT;             // NVFP4: K steps of 64 columns
};
constexpr int kAhead = 2;   // tiles of codes in flight per wavefront
constexpr int kParkBytes = 144 * 1024;

// A raw buffer load: per-lane offset and wavefront-uniform offset.  A load that
// is not wanted (past the workgroup's last tile or the wavefront's last chunk)
// reads nothing and gives zero: its lane offset lies past every buffer.  Its
// uniform offset is zero then, because the range check is made on the lane
// offset against what the uniform offset leaves of the buffer, and both
// together must stay below 2^32.
constexpr int32_t kNowhere = 0x7FFFFFFF - 64;
struct LoadAt {
  int32_t lane, uniform;
  int32_t lane_scale;   // of the block scales of the same chunk or K step
};
// LUT: `uniform` in chunks from the start of the matrix
DQ_HOST_DEVICE inline LoadAt lut_chunk_at(bool wanted, int tile, int KC, int chunk, int32_t lane, int32_t lane_scale) {
  return LoadAt{wanted ? lane : kNowhere, wanted ? tile * KC + chunk : 0, wanted ? lane_scale : kNowhere};
}
// NVFP4: a chunk's first K step in half of the 32-row tile `pair`, in bytes of
// codes from the start of the buffer
DQ_HOST_DEVICE inline int32_t nvfp4_chunk_at(bool wanted, int pair, int KT, int chunk, int half) {
  return ((pair * KT + 2 * chunk) * 1024 + half * 512) & -(int32_t)wanted;   // (no branch around the loads)
}
// and its K step `step` (h = 0 or 1), which the last chunk of an odd KT lacks
// (the scales at `uniform` / 8)
DQ_HOST_DEVICE inline LoadAt nvfp4_step_at(bool wanted, int32_t chunk_at, int step, int KT, int h, int32_t lane,
                                           int32_t lane_scale) {
  const bool in = h == 0 ? wanted : wanted && step < KT;
  return LoadAt{in ? lane : kNowhere, h == 0 ? chunk_at : (chunk_at + 1024) & -(int32_t)in, in ? lane_scale : kNowhere};
}

// K groups whose partial sums the workspace of a batch B >= 2 call holds (the
// size that callers query, and the limit of the no-allocation variant): the
// plan below uses at most these.
inline int64_t contract_groups(int64_t B, int64_t T, int64_t KC, int64_t cus) {
  const int64_t tasks = cus * (B >= 12 ? 6 : 12);
  const int64_t by_slice = std::max<int64_t>(1, (40 * 1024) / (B * 256));
  const int64_t KG = std::max<int64_t>((KC + by_slice - 1) / by_slice, std::min<int64_t>(KC, (tasks + T - 1) / T));
  const int64_t KCR = (KC + KG - 1) / KG;
  return (KC + KCR - 1) / KCR;
}

// Plan of the batch B >= 2 kernel (see lut_gemv_batch_kernel), with at most
// `most` K groups.
struct BatchedPlan {
  bool ok;                   // false: the matrix exceeds the kernel's 32-bit offsets
  int64_t BV;                // batch columns of the kernel (4, 8 or 16 >= B)
  int64_t W, CPW;            // wavefronts per workgroup, chunks per wavefront and pass
  int64_t KG, KCR, TPG, G;   // K groups, chunks per group, tiles per workgroup, workgroups
  int64_t park;              // tiles parked in LDS
};

inline bool batched_ok(int bits, int64_t T, int64_t KC) {
  if (bits == 4) return KC * 2048 * 4 < ((int64_t)1 << 31);   // (offsets within a workgroup's tiles only)
  return T * KC * 64 * (bits == 3 ? 12 : 8) < ((int64_t)1 << 31);
}

inline BatchedPlan plan_batched(int bits, int64_t B, int64_t T, int64_t KC, int64_t most, int64_t cus) {
  BatchedPlan p{};
  p.ok = batched_ok(bits, T, KC) && B * KC * 256 < ((int64_t)1 << 31);
  // sixteen wavefronts of at most three chunks (48 activation registers, of
  // the 128 that leave four wavefronts per SIMD).  Short rows take fewer
  // wavefronts and as many more workgroups per compute unit: with several
  // tiles per workgroup as few as hold the row (two or three chunks share a
  // tile's set-up: 65536 x 1056 at batch 2 14.7 -> 9.9 us), else one chunk
  // each.  More than 48 chunks: K groups, or passes over the parked tiles.
  p.BV = B > 8 ? 16 : B > 4 ? 8 : 4;
  const bool deep = T >= 2 * cus;
  p.W = deep ? (KC > 24 ? 16 : KC > 12 ? 8 : 4) : (KC > 8 ? 16 : KC > 4 ? 8 : 4);
  // but sixteen where two workgroups of eight would take two tiles each and one
  // of sixteen takes three (LUT3 10240 x 3072 at batch 2 7.8 -> 7.1 us, NVFP4
  // 10.9 -> 8.8)
  if (p.W == 8 && deep && T > 2 * cus && T <= 3 * cus) p.W = 16;
  // NVFP4 streams more bytes per chunk and gains less from the shared set-up
  // than it loses on converting x in every workgroup (batch 1, four or eight
  // against sixteen wavefronts: 18432 x 1280 8.8 / 7.7 us, 12288 x 2048 8.3 /
  // 6.6, but 24576 x 2560 11.9 / 14.1, 8192 x 1280 5.3 / 5.6, 65536 x 1056
  // 14.9 / 15.5; four against eight: 16384 x 768 6.1 / 5.5, 12288 x 768 5.0 /
  // 5.4)
  if (bits == 4 && deep) {
    if (KC > (T > 2 * cus ? 8 : 12) && (T <= (KC <= 16 ? 8 : 5) * cus || B > 8)) p.W = 16;
    else if (KC > 4 && KC <= 8 && T > 3 * cus) p.W = 8;
  }
  const int64_t fit = 3 * p.W;
  const int64_t slots = cus * (16 / p.W), fits = kParkBytes / (16 * 64 * p.BV);   // 64 W BV bytes a tile, 16 / W workgroups
  p.KG = std::min((KC + fit - 1) / fit, most);
  // chunks of the busiest wavefront over its workgroup's tiles
  auto load = [&](int64_t KG) {
    const int64_t groups = std::min<int64_t>(T, std::max<int64_t>(1, slots / KG));
    return (T + groups - 1) / groups * (((KC + KG - 1) / KG + p.W - 1) / p.W);
  };
  if (bits != 4 && p.KG > 1 && deep && T <= cus * fits && (B <= 4 || (B <= 8 && KC <= 64))) {
    // LUT, many tiles: passes need no reduction launch, and every compute unit
    // still converts each part of x once (groups against passes: 65536 x 6176
    // at batch 4 39.4 / 38.1 us, 12288 x 8192 15.2 / 13.1, 49168 x 12288 at
    // batch 2 52.1 / 47.3; at batch 8 12288 x 8192 15.2 / 13.9, but 12288 x
    // 17408 25.9 / 26.7; 5120 x 12288 at batch 2 11.8 / 12.3).  Rows just above
    // 48 chunks pay most for the second pass: 65536 x 6176 at batch 4 40.6
    // against 38.9 in the kernel with K groups staged in LDS, whose like this
    // kernel otherwise is or beats (7168 columns: 39.6 against 42.9)
    p.KG = 1;
  } else if (T * p.KG <= cus && (p.KG > 1 || (B > 8 && (KC > 40 || (KC > 32 && 3 * T <= cus))))) {
    // few tiles: more K groups use the idle compute units and leave each less
    // of x to convert, which pays for the reduction pass where there is one
    // anyway or the batch is large (batch 16: 512 x 12288 11.9 -> 8.2 us,
    // 2048 x 6144 10.1 -> 9.5; 1040 x 5120 8.8 -> 7.8, but 2048 x 4608 at
    // batch 12 7.8 / 8.3)
    p.KG = std::min(most, std::max(p.KG, std::min((KC + p.W - 1) / p.W, (B > 8 ? 2 : 1) * cus / T)));
  } else if (p.KG > 1 && p.KG < most && T * p.KG <= 4 * cus && load(p.KG + 1) <= load(p.KG)) {
    // one group more where that leaves no wavefront more to do (batch 16:
    // 2048 x 17408 14.0 -> 12.7 us, 4096 x 17408 16.9 -> 15.2, 5120 x 12288
    // 15.3 -> 14.0; with more tiles the partial sums cost more than it gives:
    // 49168 x 12288 at batch 12 53.0 / 54.0)
    ++p.KG;
  }
  p.KCR = (KC + p.KG - 1) / p.KG;
  p.KG = (KC + p.KCR - 1) / p.KCR;
  const int64_t passes = (p.KCR + fit - 1) / fit;
  p.CPW = (p.KCR + passes * p.W - 1) / (passes * p.W);
  int64_t groups = std::min<int64_t>(T, std::max<int64_t>(1, slots / p.KG));
  if (passes > 1)   // every tile stays parked over the passes: whole rounds of fuller workgroups
    groups *= (T + groups * fits - 1) / (groups * fits);
  p.TPG = (T + groups - 1) / groups;
  if (bits == 4) p.TPG = std::min(p.TPG, (((int64_t)1 << 31) - 4096) / (KC * 1024) - 2);
  p.G = (T + p.TPG - 1) / p.TPG * p.KG;
  p.park = std::min<int64_t>(p.TPG, fits);
  return p;
}

}  // namespace dq
