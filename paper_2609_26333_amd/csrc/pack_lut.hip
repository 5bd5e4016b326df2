// LUT weight packing on gfx950 (offline; the decode-side weight format).
//
// PER_ROW (benchmark decode format): one workgroup per output row finds the
// boundaries of the 2^b equal-count bins of the sorted row (by selection, not
// by sorting), sums each bin in double-double arithmetic, divides by the count
// in fp64 and rounds once to fp16 (nearest even).  Codes are the nearest entry,
// ties to the lower index, by exact comparisons with the midpoints of adjacent
// entries.
//
// PAPER_GRID (paper App. A "LUT formats"): the NVFP4 two-level scaling with a
// signed E4M3 block scale that carries the sign of the block's
// largest-magnitude element (first on ties), codes = nearest grid level of
// fp32(w / S), ties to the lower level; zero-scale blocks take the zero level.
//
// Codes are written in the 16-row x 128-column tiled layout of dq.h.
#include "dq_device.hpp"
#include "dq_internal.hpp"

namespace dq {

namespace {

// ---------------------------------------------------------------- helpers
__device__ inline uint32_t sort_key(float f) {
  uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ inline float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// Round-to-nearest-even right shift of a non-negative integer.
__device__ inline uint64_t rne_shift(uint64_t v, int s) {
  if (s <= 0) return v << (-s);
  if (s >= 64) return 0;
  const uint64_t q = v >> s;
  const uint64_t rem = v & ((1ull << s) - 1);
  const uint64_t half = 1ull << (s - 1);
  return q + ((rem > half || (rem == half && (q & 1))) ? 1 : 0);
}

// fp64 -> fp16 bits, one rounding to nearest even (finite input).
__device__ inline uint16_t f64_to_f16_rne(double d) {
  const uint64_t b = (uint64_t)__double_as_longlong(d);
  const uint16_t sign = (uint16_t)((b >> 48) & 0x8000u);
  const int exp = (int)((b >> 52) & 0x7FF);
  const uint64_t man = b & ((1ull << 52) - 1);
  if (exp == 0) return sign;                                   // zero or fp64 subnormal
  const int e = exp - 1023;
  const uint64_t full = man | (1ull << 52);
  if (e >= 16) return sign | 0x7C00u;                           // overflow
  if (e >= -14) {
    const uint64_t m = rne_shift(full, 42);                     // 11 bits, may carry to 2048
    const uint32_t h = ((uint32_t)(e + 15) << 10) + (uint32_t)(m - 1024);
    return sign | (uint16_t)(h >= 0x7C00u ? 0x7C00u : h);
  }
  // subnormal fp16: multiples of 2^-24; value = full * 2^(e - 52)
  const uint64_t m = rne_shift(full, (52 - 24) - e);
  return sign | (uint16_t)m;                                    // 1024 -> smallest normal
}

__device__ inline double f16_bits_to_f64(uint16_t h) {
  return (double)__builtin_bit_cast(_Float16, h);
}

// error-free sum
__device__ inline void two_sum(double a, double b, double& s, double& e) {
  s = a + b;
  const double bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

__device__ inline void dd_add(double& hi, double& lo, double x) {
  double s, e;
  two_sum(hi, x, s, e);
  hi = s;
  lo += e;
}

// code bits of 32 codes of one group into the dword layout of dq.h
template <int BITS>
__device__ inline void put_code(uint32_t (&w)[3], int t, uint32_t c) {
  const int s = t >> 2, b = t & 3;
  if (BITS == 3) {
    if (s < 6) {
      w[s >> 1] |= c << (8 * b + 3 * (s & 1));
    } else {
      w[s - 6] |= (c & 3u) << (8 * b + 6);
      w[2] |= (c >> 2) << (8 * b + 6 + (s - 6));
    }
  } else {
    w[s >> 2] |= c << (8 * b + 2 * (s & 3));
  }
}

template <int BITS>
__device__ inline void store_group(uint8_t* codes, int64_t row, int64_t group, int64_t KC, const uint32_t (&w)[3]) {
  constexpr int GB = BITS == 3 ? 12 : 8;
  const int64_t tile = row / 16, i = row % 16, c = group / 4, q = group % 4;
  uint32_t* p = reinterpret_cast<uint32_t*>(codes + ((tile * KC + c) * 64 + q * 16 + i) * GB);
  p[0] = w[0];
  p[1] = w[1];
  if (BITS == 3) p[2] = w[2];
}

// ---------------------------------------------------------------- PER_ROW
// One workgroup of T threads per row, the row in registers (E4 float4 per
// thread).  The equal-count bins need the row's 2^b - 1 values at the sorted
// positions j K / 2^b (thresholds T_j), not the sorted row:
//  1. a histogram of 2048 equal-width buckets over +-2.5 mean|w| (a monotone
//     map of the value, the ends open) and its prefix sums give the bucket of
//     every threshold and the class #{j : w >= T_j} of all other buckets;
//  2. each value looks its bucket up: it is added to its thread's own
//     double-double sum of its class in LDS (lane-contiguous, no bank
//     conflict), or, from a threshold's bucket (about 0.5 % of a Gaussian
//     row), goes to that bucket's list;
//  3. a wavefront ranks each threshold in its bucket's list; a crowded bucket,
//     of more than kCap members (few distinct values, extreme tails), is
//     narrowed instead: a histogram of 128 parts of the key range that holds
//     the threshold, all thresholds in one pass over the row, until one key is
//     left (no pass when the members are all equal, at most 5).  The values of these
//     buckets join the sums, which are merged in a fixed order.  Values equal to a threshold
//     that belong below it are moved by count: bin j = class j + d_{j+1}
//     T_{j+1} - d_j T_j, with d_j = j K / 2^b minus the number of values
//     below T_j (each product is exact in fp64);
//  4. codes by comparison with the midpoints rounded down to fp32 (for an
//     fp32 w the same as the exact fp64 comparison), eight lanes combining
//     their four codes each into a 32-code group.
// Bound: the VALU (77 instructions per value counted) and the LDS accesses
// beside it; the row is read once.  A bitonic sort of the row in LDS (78
// passes at K = 4096) took 1417 us for 12288 x 4096, this takes 154
// (1.4 TB/s).  Thresholds by comparison for every value, four wavefronts per
// row instead of two and a full double-double merge took 207.  Crowded rows
// (4096 x 4096, 3 bits; 461 sorted): a few distinct values 125 us, one outlier
// of 10^8 265, many octaves 255.  Bisecting each threshold by itself, bit by
// bit, took 185, 732 and 538; sixteen such rows, where a round's latency is
// all, took 155 and 123 us and now take 58 and 70 (49 sorted).  The 16 rows of
// a tile run on one XCD, so that their 12-byte groups merge into whole lines
// in its L2.
constexpr int kBuckets = 2048;
constexpr int kCap = 128;   // members of a threshold's bucket that are listed and ranked

template <int BITS, int T>
constexpr size_t pack_rows_lds() {   // the class sums; the histogram before them
  constexpr size_t sums = (size_t)(1 << BITS) * T * 16, hist = (size_t)kBuckets * 4;
  return sums > hist ? sums : hist;
}

// largest fp32 not above d
__device__ inline float f64_to_f32_down(double d) {
  const float f = (float)d;
  if (!((double)f > d)) return f;
  const uint32_t b = __float_as_uint(f);
  return __uint_as_float((b & 0x7FFFFFFFu) == 0u ? 0x80000001u : (b & 0x80000000u) ? b + 1u : b - 1u);
}

// 0 .. span in kCap equal parts or fewer: the part of x is x >> digit_shift
__device__ inline int digit_shift(uint32_t span) {
  constexpr int digit = 31 - __builtin_clz(kCap);
  static_assert(kCap == 1 << digit && kCap == 128, "two parts per lane");
  return max(0, 32 - digit - __builtin_clz(span | 1u));
}

// #{j : x > m[j]}, m ascending
template <int NT>
__device__ inline uint32_t code_of(float x, const float (&m)[NT]) {
  if constexpr (NT == 7) {
    const bool b2 = x > m[3];
    const bool b1 = x > (b2 ? m[5] : m[1]);
    const float lo = b1 ? m[2] : m[0], hi = b1 ? m[6] : m[4];
    const bool b0 = x > (b2 ? hi : lo);
    return (b2 ? 4u : 0u) + (b1 ? 2u : 0u) + (b0 ? 1u : 0u);
  } else {
    const bool b1 = x > m[1];
    const bool b0 = x > (b1 ? m[2] : m[0]);
    return (b1 ? 2u : 0u) + (b0 ? 1u : 0u);
  }
}

template <int BITS, int T, int E4>
__global__ __launch_bounds__(T) void pack_lut_per_row_kernel(const float* __restrict__ W, int64_t N, int64_t tiles,
                                                             int K, int KC, uint8_t* __restrict__ codes,
                                                             uint16_t* __restrict__ lut) {
  constexpr int NB = 1 << BITS, NT = NB - 1, NW = T / 64, BPT = kBuckets / T;
  constexpr int GB = BITS == 3 ? 12 : 8;
  extern __shared__ __align__(16) uint8_t smem[];
  uint32_t* hist = reinterpret_cast<uint32_t*>(smem);
  double2* sums = reinterpret_cast<double2*>(smem);          // [NB][T], once the histogram has been scanned
  // class, or the bucket's first threshold + 0x80 (listed) or + 0xC0 (crowded)
  __shared__ uint8_t s_mark[kBuckets];
  __shared__ uint32_t s_cand[NT][kCap];
  __shared__ float s_f[NW];
  __shared__ uint32_t s_w[2][NW];
  __shared__ int s_slot[NT], s_lo[NT], s_cnt[NT], s_fill[NT], s_less[NT];
  __shared__ uint4 s_range[NT + 1];
  __shared__ uint32_t s_key[NT], s_span[NT], s_min[NT], s_max[NT];
  __shared__ double s_hi[NB], s_lo2[NB];
  __shared__ uint16_t s_entry[NB];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // workgroup b runs on XCD b % 8: tile = 8 (b / 128) + b % 8, row (b / 8) % 16 of it
  const int64_t tile = (int64_t)(blockIdx.x >> 7) * 8 + (blockIdx.x & 7);
  if (tile >= tiles) return;
  const int ri = (int)((blockIdx.x >> 3) & 15);
  const int64_t row = tile * 16 + ri;
  const int sub = tid & 7;
  // dword `sub` of group g of this row
  auto code_dword = [&](int g) {
    return reinterpret_cast<uint32_t*>(codes + ((tile * KC + (g >> 2)) * 64 + (g & 3) * 16 + ri) * GB) + sub;
  };
  if (row >= N) {   // padding rows of the last 16-row tile: zero codes and entries
    for (int q = tid; q < KC * 32; q += T)
      if (sub < GB / 4) *code_dword(q >> 3) = 0u;
    if (tid < NB) lut[row * NB + tid] = 0;
    return;
  }

  // ---- the row (quad q = tid + e T: columns 4q .. 4q + 3), sum |w|
  const float4_t* wr = reinterpret_cast<const float4_t*>(W + row * K);
  const int nq = K / 4;   // K % 32 == 0
  float v[E4][4];
  float s = 0.0f;
#pragma unroll
  for (int e = 0; e < E4; ++e) {
    const int q = tid + e * T;
    const float4_t x = q < nq ? wr[q] : float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) v[e][t] = x[t];
  }
#pragma unroll
  for (int i = 0; i < BPT; ++i) hist[tid + i * T] = 0u;
#pragma unroll
  for (int e = 0; e < E4; ++e)
#pragma unroll
    for (int t = 0; t < 4; ++t) s += fabsf(v[e][t]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) s_f[wave] = s;
  if (tid < NT) {
    s_slot[tid] = s_lo[tid] = s_less[tid] = 0;
    s_cnt[tid] = s_fill[tid] = 0;
    s_key[tid] = s_span[tid] = s_max[tid] = 0u;
    s_min[tid] = 0xFFFFFFFFu;
  }
  __syncthreads();
  float total = 0.0f;
#pragma unroll
  for (int w = 0; w < NW; ++w) total += s_f[w];
  const float scale = fminf(1e30f, (kBuckets / 5.0f) / (total / (float)K));
  auto bucket = [&](float x) {   // non-decreasing in x
    return (int)__builtin_amdgcn_fmed3f(__builtin_fmaf(x, scale, 0.5f * kBuckets), 0.0f, (float)(kBuckets - 1));
  };

  // ---- 1. histogram, prefix sums, marks
#pragma unroll
  for (int e = 0; e < E4; ++e)
    if (tid + e * T < nq)
#pragma unroll
      for (int t = 0; t < 4; ++t) atomicAdd(&hist[bucket(v[e][t])], 1u);
  __syncthreads();
  const int cnt = K / NB;
  {
    uint32_t h[BPT];
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) mine += h[i] = hist[tid * BPT + i];
    uint32_t incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t o = (uint32_t)__shfl_up((int)incl, off, 64);
      if (lane >= off) incl += o;
    }
    if (lane == 63) s_w[0][wave] = incl;
    __syncthreads();
    uint32_t lo = incl - mine;
    for (int w = 0; w < wave; ++w) lo += s_w[0][w];
    int j = 1;   // the next threshold at or past this position
    while (j <= NT && (uint32_t)(j * cnt) < lo) ++j;
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      uint32_t mark = (uint32_t)(j - 1);   // thresholds below the bucket
      const int first = j;
      for (; j <= NT && (uint32_t)(j * cnt) < lo + h[i]; ++j) {
        mark = (h[i] > (uint32_t)kCap ? 0xC0u : 0x80u) + (uint32_t)(first - 1);
        s_slot[j - 1] = first - 1;
        s_lo[j - 1] = (int)lo;
        s_less[j - 1] = (int)lo;
        s_cnt[j - 1] = (int)h[i];
      }
      s_mark[tid * BPT + i] = (uint8_t)mark;
      lo += h[i];
    }
  }
  __syncthreads();

  // ---- 2. class sums, and the members of the marked buckets
#pragma unroll
  for (int c = 0; c < NB; ++c) sums[c * T + tid] = double2{0.0, 0.0};
  auto add = [&](int c, float x) {
    double2 a = sums[c * T + tid];
    dd_add(a.x, a.y, (double)x);
    sums[c * T + tid] = a;
  };
#pragma unroll
  for (int e = 0; e < E4; ++e)
    if (tid + e * T < nq)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const uint32_t m = s_mark[bucket(v[e][t])];
        if (m & 0x80u) {
          const uint32_t key = sort_key(v[e][t]);
          if (m & 0x40u) {
            atomicMin(&s_min[m & 7u], key);
            atomicMax(&s_max[m & 7u], key);
          } else {
            const int p = atomicAdd(&s_fill[m & 7u], 1);
            if (p < kCap) s_cand[m & 7u][p] = key;   // always, for finite values
          }
        }
        add((int)(m & 7u), (m & 0x80u) ? 0.0f : v[e][t]);
      }
  __syncthreads();

  // ---- 3. thresholds
  bool listed = true;   // every marked bucket fits its list
  for (int j = 0; j < NT; ++j) listed = listed && s_cnt[j] <= kCap;
  for (int j = wave; j < NT; j += NW) {
    const int n = s_cnt[j], rank = (j + 1) * cnt - s_lo[j];
    if (n > kCap) continue;
    const uint32_t* c = s_cand[s_slot[j]];
    for (int c0 = 0; c0 < n; c0 += 64) {
      const bool in = c0 + lane < n;
      const uint32_t key = in ? c[c0 + lane] : 0u;
      int less = 0, same = 0;
      for (int i = 0; i < n; ++i) {
        const uint32_t o = c[i];
        less += o < key ? 1 : 0;
        same += o == key ? 1 : 0;
      }
      if (in && less <= rank && rank < less + same) {   // every lane that holds the value
        s_key[j] = key;
        s_less[j] = s_lo[j] + less;
      }
    }
  }
  if (!listed) {
    // the range base .. base + span of keys of the bucket that holds threshold j
    if (tid < NT && s_cnt[tid] > kCap) {
      s_key[tid] = s_min[s_slot[tid]];
      s_span[tid] = s_max[s_slot[tid]] - s_key[tid];
    }
    __syncthreads();
    for (int round = 0; round < 5; ++round) {   // each leaves 7 bits less of the ranges
      // the distinct ranges in ascending order (equal bases: equal ranges; two
      // that differ have no key in common), each with a row of counts
      uint32_t base[NT], rows = 0u;
      int n = 0;
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const uint32_t b = s_key[j], span = s_span[j];
        base[j] = 0xFFFFFFFFu;
        if (span != 0u && (n == 0 || b != s_key[j - 1] || s_span[j - 1] == 0u)) {
          if (tid == 0) s_range[n + 1] = uint4{b, span, (uint32_t)digit_shift(span), (uint32_t)j};
          ++n;
          rows |= 1u << j;
          if (tid < kCap) s_cand[j][tid] = 0u;
        }
      }
      if (n == 0) break;
      if (tid == 0) s_range[0] = uint4{0xFFFFFFFFu, 0u, 0u, 0u};   // keys below the first: none
      __syncthreads();
#pragma unroll
      for (int j = 0; j < NT; ++j)
        if (j < n) base[j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_range[j + 1].x);
#pragma unroll
      for (int e = 0; e < E4; ++e) {
        if (tid + e * T < nq)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            float x = v[e][t];
            asm volatile("" : "+v"(x));   // the keys of the row are not kept from round to round: registers
            const uint32_t key = sort_key(x);
            int i = 0;
#pragma unroll
            for (int j = 0; j < NT; ++j) i += key >= base[j] ? 1 : 0;
            const uint4 r = s_range[min(i, n)];
            if (key - r.x <= r.y) atomicAdd(&s_cand[r.w][(key - r.x) >> r.z], 1u);
          }
        __builtin_amdgcn_sched_barrier(0);   // no table entries in flight for the next quad either
      }
      __syncthreads();
      for (int j = wave; j < NT; j += NW) {
        const uint32_t from = s_key[j], span = s_span[j];
        if (span == 0u) continue;
        const int row_of = 31 - __clz((int)(rows & ((2u << j) - 1u)));
        const uint32_t h0 = s_cand[row_of][2 * lane], h1 = s_cand[row_of][2 * lane + 1];
        uint32_t hi = h0 + h1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const uint32_t o = (uint32_t)__shfl_up((int)hi, off, 64);
          if (lane >= off) hi += o;
        }
        const uint32_t lo = hi - h0 - h1, rank = (uint32_t)((j + 1) * cnt - s_less[j]);
        if (lo <= rank && rank < hi) {   // one lane
          const bool second = rank >= lo + h0;
          const int shift = digit_shift(span);
          const uint32_t to = from + ((uint32_t)(2 * lane + (second ? 1 : 0)) << shift);
          s_key[j] = to;
          s_span[j] = min((1u << shift) - 1u, from + span - to);
          s_less[j] += (int)(lo + (second ? h0 : 0u));
        }
      }
      __syncthreads();
    }
  }
  __syncthreads();
  // the members of the marked buckets join their classes
  auto class_of = [&](uint32_t key) {
    int c = 0;
#pragma unroll
    for (int j = 0; j < NT; ++j) c += key >= s_key[j] ? 1 : 0;
    return c;
  };
  for (int j = wave; j < NT; j += NW) {
    const int n = s_cnt[j];
    if (s_slot[j] != j || n > kCap) continue;
    for (int i = lane; i < n; i += 64) add(class_of(s_cand[j][i]), key_value(s_cand[j][i]));
  }
  if (!listed) {
#pragma unroll
    for (int e = 0; e < E4; ++e)
      if (tid + e * T < nq)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const uint32_t m = s_mark[bucket(v[e][t])];
          if (m & 0x40u) add(class_of(sort_key(v[e][t])), v[e][t]);
        }
  }
  __syncthreads();
  // the T sums of a class: LPB lanes take T / LPB each, then a butterfly
  // (sums of the high parts without error, their errors with the low parts)
  constexpr int LPB = T / NB < 64 ? T / NB : 64;
  if (tid < NB * LPB) {
    const int c = tid / LPB, l = tid % LPB;
    double2 a = sums[c * T + l];
#pragma unroll
    for (int i = 1; i < T / LPB; ++i) {
      const double2 o = sums[c * T + LPB * i + l];
      dd_add(a.x, a.y, o.x);
      a.y += o.y;
    }
#pragma unroll
    for (int off = LPB / 2; off >= 1; off >>= 1) {
      const double h = __shfl_xor(a.x, off, 64), o = __shfl_xor(a.y, off, 64);
      dd_add(a.x, a.y, h);
      a.y += o;
    }
    if (l == 0) {
      s_hi[c] = a.x;
      s_lo2[c] = a.y;
    }
  }
  __syncthreads();
  if (tid < NB) {
    double h = s_hi[tid], l = s_lo2[tid];
    if (tid < NT) dd_add(h, l, (double)((tid + 1) * cnt - s_less[tid]) * (double)key_value(s_key[tid]));
    if (tid > 0) dd_add(h, l, -((double)(tid * cnt - s_less[tid - 1]) * (double)key_value(s_key[tid - 1])));
    const uint16_t entry = f64_to_f16_rne((h + l) / (double)cnt);
    s_entry[tid] = entry;
    lut[row * NB + tid] = entry;
  }
  __syncthreads();

  // ---- 4. codes
  float mid[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
    mid[j] = f64_to_f32_down((f16_bits_to_f64(s_entry[j]) + f16_bits_to_f64(s_entry[j + 1])) * 0.5);
  const int l0 = lane & ~7;
#pragma unroll
  for (int e = 0; e < E4; ++e) {
    const int q = tid + e * T, g = q >> 3;   // q % 8 == sub: the quad's place in its group
    uint32_t sel = 0u;
    if (q < nq) {
#pragma unroll
      for (int t = 0; t < 4; ++t) sel |= code_of<NT>(v[e][t], mid) << (8 * t);
    }
    if constexpr (BITS == 3) {
      const int p = l0 + 2 * min(sub, 2);
      const uint32_t a = (uint32_t)__shfl((int)sel, p, 64), b = (uint32_t)__shfl((int)sel, p + 1, 64);
      const uint32_t s6 = (uint32_t)__shfl((int)sel, l0 + 6, 64), s7 = (uint32_t)__shfl((int)sel, l0 + 7, 64);
      uint32_t w = a | (b << 3);
      w |= sub == 0 ? (s6 & 0x03030303u) << 6
           : sub == 1 ? (s7 & 0x03030303u) << 6
                      : ((s6 & 0x04040404u) << 4) | ((s7 & 0x04040404u) << 5);
      if (sub < 3 && g < KC * 4) *code_dword(g) = w;
    } else {
      uint32_t w = sel << (2 * (sub & 3));
      w |= (uint32_t)__shfl_xor((int)w, 1, 64);
      w |= (uint32_t)__shfl_xor((int)w, 2, 64);
      if ((sub & 3) == 0 && g < KC * 4) code_dword(g)[(sub >> 2) - sub] = w;
    }
  }
}

// Threads and float4 per thread for rows of K: as few wavefronts as hold the
// row in registers, since the scan and the merges are per-thread work.
template <int BITS>
hipError_t launch_pack_rows(const float* W, int64_t N, int64_t K, const LutView& out, hipStream_t s) {
  typedef void (*kern_t)(const float*, int64_t, int64_t, int, int, uint8_t*, uint16_t*);
  struct Pick {
    int64_t cols;
    kern_t kern;
    int threads;
    size_t lds;
  };
#define DQ_PACK_ROWS(T, E4) \
  Pick { (int64_t)T * E4 * 4, pack_lut_per_row_kernel<BITS, T, E4>, T, pack_rows_lds<BITS, T>() }
  static const Pick picks[] = {DQ_PACK_ROWS(128, 2), DQ_PACK_ROWS(128, 4), DQ_PACK_ROWS(128, 8), DQ_PACK_ROWS(128, 10),
                               DQ_PACK_ROWS(256, 8), DQ_PACK_ROWS(512, 6), DQ_PACK_ROWS(512, 9),
                               DQ_PACK_ROWS(1024, 6), DQ_PACK_ROWS(1024, 8)};
#undef DQ_PACK_ROWS
  const Pick* p = picks;
  while (p->cols < K) ++p;   // K <= 32768
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(p->kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)p->lds);
  if (e != hipSuccess) return e;
  const int64_t tiles = round_up(N, 16) / 16;
  hipLaunchKernelGGL(p->kern, dim3((unsigned)(round_up(tiles, 8) * 16)), dim3(p->threads), p->lds, s, W, N, tiles,
                     (int)K, (int)(round_up(K, 128) / 128), out.codes, out.lut);
  return hipGetLastError();
}

// ---------------------------------------------------------------- PAPER_GRID
struct Grid {
  uint16_t v[8];
};

template <int BITS>
__global__ __launch_bounds__(256) void pack_lut_paper_kernel(const float* __restrict__ W, int64_t N, int64_t N16,
                                                             int64_t K, int64_t KC, const float* __restrict__ Gp,
                                                             Grid grid, int zero_level, uint8_t* __restrict__ codes,
                                                             uint8_t* __restrict__ scales, uint16_t* __restrict__ lut_out) {
  constexpr int NL = 1 << BITS;
  const int64_t groups = KC * 4;
  const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (gid < NL) lut_out[gid] = grid.v[gid];
  if (gid >= N16 * groups) return;
  const int64_t row = gid / groups, g = gid % groups;
  double mid[NL - 1];
#pragma unroll
  for (int m = 0; m < NL - 1; ++m) mid[m] = (f16_bits_to_f64(grid.v[m]) + f16_bits_to_f64(grid.v[m + 1])) * 0.5;
  const float G = *Gp;
  uint32_t w[3] = {0u, 0u, 0u};
  uint32_t sb[2] = {0u, 0u};
  for (int h = 0; h < 2; ++h) {
    const int64_t k0 = g * 32 + h * 16;
    if (row >= N || k0 >= K) continue;           // padding: code 0, scale 0
    const float* wp = W + row * K + k0;
    float best = wp[0];
    float amax = fabsf(best);
    for (int t = 1; t < 16; ++t) {
      const float a = fabsf(wp[t]);
      if (a > amax) {
        amax = a;
        best = wp[t];
      }
    }
    const float t_ = amax / (6.0f * G);
    const uint32_t mag = e4m3_encode_rne_sat(t_);
    const uint32_t sbyte = mag | ((best < 0.0f && mag != 0u) ? 0x80u : 0u);
    const float S = e4m3_decode(sbyte) * G;
    sb[h] = sbyte;
    for (int t = 0; t < 16; ++t) {
      uint32_t c;
      if (S == 0.0f) {
        c = (uint32_t)zero_level;
      } else {
        const double y = (double)(wp[t] / S);
        c = 0;
#pragma unroll
        for (int m = 0; m < NL - 1; ++m) c += y > mid[m] ? 1u : 0u;
      }
      put_code<BITS>(w, h * 16 + t, c);
    }
  }
  store_group<BITS>(codes, row, g, KC, w);
  const int64_t tile = row / 16, i = row % 16, c = g / 4, q = g % 4;
  uint8_t* sp = scales + (tile * KC + c) * 128 + (q * 16 + i) * 2;
  sp[0] = (uint8_t)sb[0];
  sp[1] = (uint8_t)sb[1];
}

// ---------------------------------------------------------------- autocast
// LUT -> NVFP4 autocast, step 1: the dequantized LUT weight as fp32 [N, K],
// one thread per 32-code group of the tiled layout (dq.h).  PER_ROW entries
// are fp16 (exact in fp32); a PAPER_GRID value grid * e4m3 * G is computed
// as fp32(grid * e4m3) (exact: at most 15 significant bits) times G, one
// rounding of the exact product.
template <int BITS, int MODE>
__global__ __launch_bounds__(256) void lut_dequant_kernel(const uint8_t* __restrict__ codes,
                                                          const uint16_t* __restrict__ lut,
                                                          const uint8_t* __restrict__ scales,
                                                          const float* __restrict__ Gp, int64_t N, int64_t K,
                                                          int64_t tiles_c, float* __restrict__ out) {
  constexpr int GB = BITS == 3 ? 12 : 8;   // bytes per 32-code group
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t tile = gid >> 6;
  const int g = (int)(gid & 63), i = g & 15, q = g >> 4;
  const int64_t tr = tile / tiles_c, c = tile - tr * tiles_c;
  const int64_t row = tr * 16 + i, col0 = c * 128 + q * 32;
  if (row >= N || col0 >= K) return;
  const uint8_t* gp = codes + tile * 64 * GB + g * GB;
  uint32_t d[3];
  d[0] = *reinterpret_cast<const uint32_t*>(gp);
  d[1] = *reinterpret_cast<const uint32_t*>(gp + 4);
  d[2] = BITS == 3 ? *reinterpret_cast<const uint32_t*>(gp + 8) : 0u;
  float sb[2] = {1.0f, 1.0f};
  float G = 1.0f;
  if (MODE == 1) {
    sb[0] = e4m3_decode(scales[tile * 128 + g * 2]);
    sb[1] = e4m3_decode(scales[tile * 128 + g * 2 + 1]);
    G = *Gp;
  }
  float* o = out + row * K + col0;
#pragma unroll
  for (int t = 0; t < 32; ++t) {
    const int sl = t >> 2, b = t & 3;
    uint32_t code;
    if (BITS == 3) {
      if (sl < 6)
        code = (d[sl >> 1] >> (8 * b + 3 * (sl & 1))) & 7u;
      else
        code = ((d[sl - 6] >> (8 * b + 6)) & 3u) | (((d[2] >> (8 * b + 6 + (sl - 6))) & 1u) << 2);
    } else {
      code = (d[sl >> 2] >> (8 * b + 2 * (sl & 3))) & 3u;
    }
    const uint16_t e = MODE == 0 ? lut[row * (1 << BITS) + code] : lut[code];
    const float v = (float)__builtin_bit_cast(_Float16, e);
    if (MODE == 0) {
      o[t] = v;
    } else {
      const float p = v * sb[t >> 4];   // exact
      o[t] = p * G;
    }
  }
}

}  // namespace

// paper grids (App. A "LUT formats") rounded to fp16
static const uint16_t kPaperLut3[8] = {0xC4B4, 0xC1BD, 0xBD7A, 0x0000, 0x3CE2, 0x410F, 0x440C, 0x4600};
static const uint16_t kPaperLut2[4] = {0xC34E, 0x0000, 0x410C, 0x4600};

const uint16_t* paper_grid_fp16(int bits) { return bits == 3 ? kPaperLut3 : kPaperLut2; }

hipError_t launch_pack_lut(const float* W, int64_t N, int64_t K, const uint16_t* grid_host, const LutView& out,
                           hipStream_t s) {
  const int64_t N16 = round_up(N, 16), KC = round_up(K, 128) / 128;
  if (N16 == 0) return hipSuccess;
  if (out.mode == 0) {
    return out.bits == 3 ? launch_pack_rows<3>(W, N, K, out, s) : launch_pack_rows<2>(W, N, K, out, s);
  }
  const int NL = 1 << out.bits;
  Grid g{};
  const uint16_t* src = grid_host ? grid_host : paper_grid_fp16(out.bits);
  int zl = -1;
  for (int i = 0; i < NL; ++i) {
    g.v[i] = src[i];
    if ((src[i] & 0x7FFFu) == 0) zl = i;
  }
  hipError_t e = launch_global_scale_f32(W, N * K, out.G, s);   // G = max|W| / 2688, the NVFP4 rule
  if (e != hipSuccess) return e;
  const int64_t threads = N16 * KC * 4;
  const int64_t blocks = (threads + 255) / 256;
  if (out.bits == 3)
    hipLaunchKernelGGL(pack_lut_paper_kernel<3>, dim3((unsigned)blocks), dim3(256), 0, s, W, N, N16, K, KC, out.G, g,
                       zl, out.codes, out.scales, out.lut);
  else
    hipLaunchKernelGGL(pack_lut_paper_kernel<2>, dim3((unsigned)blocks), dim3(256), 0, s, W, N, N16, K, KC, out.G, g,
                       zl, out.codes, out.scales, out.lut);
  return hipGetLastError();
}

hipError_t launch_autocast_lut(const LutView& w, const float* G_override, const NvFp4View& out, hipStream_t s) {
  const int64_t N = w.rows, K = w.cols;
  float* tmp = nullptr;
  hipError_t e = hipSuccess;
  if (N * K > 0) {
    e = pool_alloc_async(reinterpret_cast<void**>(&tmp), (size_t)(N * K) * 4, s);
    if (e != hipSuccess) return e;
    const int64_t tiles_c = (K + 127) / 128;
    const int64_t threads = (N + 15) / 16 * tiles_c * 64;
    typedef void (*kern_t)(const uint8_t*, const uint16_t*, const uint8_t*, const float*, int64_t, int64_t, int64_t,
                           float*);
    const kern_t kern = w.bits == 3 ? (w.mode == 0 ? lut_dequant_kernel<3, 0> : lut_dequant_kernel<3, 1>)
                                    : (w.mode == 0 ? lut_dequant_kernel<2, 0> : lut_dequant_kernel<2, 1>);
    hipLaunchKernelGGL(kern, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, w.codes, w.lut, w.scales, w.G,
                       N, K, tiles_c, tmp);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = launch_pack_nvfp4(tmp, N, K, G_override, out, s);
  if (tmp != nullptr) {
    const hipError_t f = hipFreeAsync(tmp, s);
    if (e == hipSuccess) e = f;
  }
  return e;
}

}  // namespace dq
