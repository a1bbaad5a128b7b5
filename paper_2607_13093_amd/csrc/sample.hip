// Temperature + top-p sampling of each verification row, then the accepted
// draft prefix of each session (eq. 15 with a nucleus cut; Section 5.5).
//
// One 512-thread block per row of fused logits f (fp32, written by the
// endpoint projection, whose per-tile argmax keys also give the row maximum).
// The row is walked in chunks of 256 positions, one per wave iteration (lane
// l holds positions 4l .. 4l+3 of the chunk, loaded as one 16-byte vector),
// so every pass is a short rolled loop of coalesced loads.
//
// Weights.  e = exp((f - fmax) / tau) in fp64 by the table-driven method of
// Tang (ACM TOMS 15(2), 1989): with t = (f - fmax) / (tau ln2) * 256,
// N = rint(t), r = t - N (|r| <= 1/2), e = 2^(N>>8) * 2^((N&255)/256) * 2^(r/256),
// the middle factor from a 256-entry table and 2^(r/256) a degree-4 Taylor
// polynomial (truncation below 4e-17).  Every use of a weight evaluates the
// same operations with contraction off, so it is bit-identical wherever it is
// recomputed.
//
// Exact masses.  Each weight e in [0, 1] becomes E = floor(e * 2^56), the
// mantissa of the product of table entry and polynomial shifted into place.
// Masses are exact integer sums of E (added as E = a * 2^28 + b), so the
// nucleus cut and the inverse CDF are exact for these weights, independent of
// summation order, and the kernel is deterministic.  E misses e * 2^56 by less
// than one unit.
//
// The passes are bound by their instructions (65536 positions keep a CU's
// SIMDs busy for 31 us in the exact pass, of 61): N comes out of the low word
// of t + 1.5 * 2^52 and E out of shifts, as rounding to and converting from
// fp64 are quarter-rate operations, and pass 1 counts elements instead of
// adding weights.
//
//   1. A histogram of element counts over 4096 value buckets of
//      y = (fmax - f)/tau in [0, 24) (the last bucket also takes y >= 24, whose
//      elements each weigh below 4e-11); a bucket's mass is estimated as its
//      count times the weight of its middle.  Bucket order is value order, so
//      the nucleus -- the shortest prefix of (p desc, id asc) reaching
//      top_p * Z -- ends near the bucket where the running estimate reaches
//      top_p of the total.  The window is every bucket that may hold the cut,
//      given how far off the estimate can be (pick_window); where those have
//      more elements than the list, fewer buckets around the estimate.
//   2. One exact pass: Z; the masses of the buckets below the window, per
//      segment (runs of consecutive positions, at most 512 per row); the
//      window's elements into an LDS list.  An exact histogram of the list
//      over 128 sub-buckets per bucket finds the sub-bucket holding the cut;
//      one wave ranks its few elements by (key desc, position asc) to find
//      the element completing the nucleus.  The nucleus is
//      {key > T} + {key == T, position <= cut}.
//      Should a narrowed window miss the cut or overflow the list, the pass is
//      redone on its neighbours, then an exact histogram over groups of 4
//      buckets picks the group and the pass is redone on it; a sub-bucket holding more than 64 elements is ranked by
//      a bitonic sort of the list, and a group with more than 1024 elements
//      goes through an exact radix select over its keys (8 bits per pass),
//      the cut among elements tied at the threshold key being the c-th in id
//      order.
//   3. u = top 24 bits of word 0 of Philox4x32-10 (key = seed halves,
//      counter = (row in session, session, 0, 0)).  The token is the first
//      nucleus member in id order whose running mass M has
//      M * 2^24 > u24 * mass(nucleus): a scan over segment masses picks the
//      segment, one wave scans inside it.
#include <algorithm>

#include "sph_internal.h"

namespace sph {

constexpr int kSThreads = 512;
constexpr int kSWaves = kSThreads / 64;
constexpr int kBuckets = 4096;     // value buckets of (fmax - f)/tau over [0, kYSpan)
constexpr int kBPT = kBuckets / kSThreads;
constexpr int kCoarse = 1024;      // exact fallback histogram: 4 value buckets each
constexpr int kSub = 128;          // sub-buckets per bucket of the window
constexpr int kMaxSub = 4 * kSub;  // sub-buckets of a window (coarser ones past 4 buckets)
constexpr int kMaxSeg = kSThreads; // segments per row, one per thread in scans
constexpr int kMaxCand = 1024;     // window elements held in LDS
constexpr int kChunk = 256;        // positions per wave iteration
constexpr int kSegChunks = 4;      // chunks per segment at least
constexpr float kYSpan = 24.0f;
static_assert(kMaxCand == 2 * kSThreads, "two list entries per thread");
static_assert(kCoarse == 2 * kSThreads, "two coarse buckets per thread");
static_assert(kMaxSub == kSThreads, "one sub-bucket per thread");

// 2^(r/256) = exp(r * ln2/256): Taylor coefficients (ln2/256)^k / k!
constexpr int kTab = 256;
constexpr double kLn2 = 0.6931471805599453;
constexpr double kL = kLn2 / kTab;
constexpr double kC1 = kL;
constexpr double kC2 = kL * kL / 2.0;
constexpr double kC3 = kL * kL * kL / 6.0;
constexpr double kC4 = kL * kL * kL * kL / 24.0;

// ---------------------------------------------------------------------------
// 128-bit unsigned integers (masses in units of 2^-56)

struct U128 {
  uint64_t lo, hi;
};

__device__ __forceinline__ U128 u128_add(U128 a, U128 b) {
  U128 r;
  r.lo = a.lo + b.lo;
  r.hi = a.hi + b.hi + (r.lo < a.lo ? 1ull : 0ull);
  return r;
}

__device__ __forceinline__ U128 u128_sub(U128 a, U128 b) {
  U128 r;
  r.lo = a.lo - b.lo;
  r.hi = a.hi - b.hi - (a.lo < b.lo ? 1ull : 0ull);
  return r;
}

__device__ __forceinline__ bool u128_lt(U128 a, U128 b) {
  return a.hi < b.hi || (a.hi == b.hi && a.lo < b.lo);
}

__device__ __forceinline__ U128 u128_shl24(U128 a) {
  return U128{a.lo << 24, (a.hi << 24) | (a.lo >> 40)};
}

__device__ __forceinline__ U128 u128_mul32(U128 a, uint32_t m) {
  return U128{a.lo * m, a.hi * m + __umul64hi(a.lo, (uint64_t)m)};
}

// A * 2^28 + B
__device__ __forceinline__ U128 u128_join(uint64_t A, uint64_t B) {
  return u128_add(U128{A << 28, A >> 36}, U128{B, 0ull});
}

__device__ __forceinline__ double u128_to_f64(U128 a) {
  return (double)a.hi * 0x1.0p64 + (double)a.lo;
}

// ceil(x) for finite x >= 0 (x < 2^127)
__device__ U128 u128_ceil(double x) {
  if (!(x > 0.0)) return U128{0ull, 0ull};
  if (x < 1.0) return U128{1ull, 0ull};
  const uint64_t bits = (uint64_t)__double_as_longlong(x);
  const int e = (int)(bits >> 52) - 1023;
  const uint64_t m = (bits & 0xFFFFFFFFFFFFFull) | 0x10000000000000ull;  // x = m * 2^(e-52)
  if (e <= 52) {
    const int sh = 52 - e;
    uint64_t q = m >> sh;
    if ((q << sh) != m) ++q;
    return U128{q, 0ull};
  }
  const int sh = e - 52;
  if (sh < 64) return U128{m << sh, m >> (64 - sh)};
  return U128{0ull, m << (sh - 64)};
}

// The two parts that a sum of E is accumulated in.
constexpr uint32_t kLow28 = (1u << 28) - 1u;
__device__ __forceinline__ uint64_t part_a(uint64_t e) { return e >> 28; }
__device__ __forceinline__ uint64_t part_b(uint64_t e) { return (uint32_t)e & kLow28; }

// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t orderable(float v) {
  v = v + 0.0f;  // -0 -> +0
  const uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float from_orderable(uint32_t k) {
  const uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
  return __uint_as_float(u);
}

// floor(exp((x - fmax) / tau) * 2^56) with kk = kTab / (tau ln2), c0 = -fmax * kk.
__device__ __forceinline__ uint64_t weight56(float x, double kk, double c0,
                                             const double* __restrict__ tab) {
#pragma clang fp contract(off)
  double t = fma((double)x, kk, c0);
  t = fmin(fmax(t, -58.0 * kTab), 0.0);  // below 2^-57 the result is 0; x <= fmax
  const double s = t + 0x1.8p52;         // rint(t) in the low word
  const int j = (int)(uint32_t)__double_as_longlong(s);
  const double r = t - (s - 0x1.8p52);   // exact, |r| <= 1/2
  const double p = fma(r, fma(r, fma(r, fma(r, kC4, kC3), kC2), kC1), 1.0);
  // in [0.998, 1.998): exponent 0 or -1
  const uint64_t q = (uint64_t)__double_as_longlong(tab[j & (kTab - 1)] * p);
  const int e = (int)(q >> 52) - 1023 + (j >> 8);  // of the weight, in [-59, 0]
  const uint64_t m = (q & 0xFFFFFFFFFFFFFull) | 0x10000000000000ull;  // weight = m * 2^(e - 52)
  return (m << 4) >> (-e);
}

// (fmax - x) * kb with kb = kBuckets / (kYSpan tau): bucket units, >= 0.
__device__ __forceinline__ float ypos(float x, float vmax, float kb) {
#pragma clang fp contract(off)
  return (vmax - x) * kb;
}

// Value bucket: floor(ypos), the last bucket taking everything beyond.
// Non-decreasing as x decreases.
__device__ __forceinline__ int bucket_of(float y) {
  return (int)fminf(y, (float)(kBuckets - 1));
}

// Sub-bucket: floor(ypos * kSub) (exact scaling), consistent with bucket_of:
// bucket b holds sub-buckets [kSub b, kSub b + kSub - 1].
__device__ __forceinline__ int subbucket_of(float y) {
  return (int)fminf(y * (float)kSub, (float)(kSub * kBuckets - 1));
}

// Philox4x32-10 (Salmon et al., SC'11), word 0 of the output block.
__device__ uint32_t philox_x0(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                              uint32_t k1) {
  constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
  constexpr uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += W0;
      k1 += W1;
    }
    const uint32_t hi0 = __umulhi(M0, c0), lo0 = M0 * c0;
    const uint32_t hi1 = __umulhi(M1, c2), lo1 = M1 * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  return c0;
}

// ---------------------------------------------------------------------------
// wave and block primitives (fixed order)

// Sum over the wave, in every lane, without the LDS crossbar: the 32- and
// 16-lane steps swap register halves with v_permlane32_swap /
// v_permlane16_swap (both results summed), then DPP rotations by 8, 4, 2
// and 1 lanes inside each 16-lane row finish the sum.
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
  return ((uint64_t)dpp_u32<CTRL>((uint32_t)(v >> 32)) << 32) | dpp_u32<CTRL>((uint32_t)v);
}
template <bool W32>
__device__ __forceinline__ uint64_t swap_sum_u64(uint64_t v) {
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  const auto l = W32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                     : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto h = W32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                     : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return (((uint64_t)h[0] << 32) | l[0]) + (((uint64_t)h[1] << 32) | l[1]);
}
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
  v = swap_sum_u64<true>(v);
  v = swap_sum_u64<false>(v);
  v += dpp_u64<0x128>(v);  // row_ror:8
  v += dpp_u64<0x124>(v);  // row_ror:4
  v += dpp_u64<0x122>(v);  // row_ror:2
  v += dpp_u64<0x121>(v);  // row_ror:1
  return v;
}

// Maximum over the wave, in every lane, by the same moves.
template <bool W32>
__device__ __forceinline__ uint64_t swap_max_u64(uint64_t v) {
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  const auto l = W32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                     : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto h = W32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                     : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return max(((uint64_t)h[0] << 32) | l[0], ((uint64_t)h[1] << 32) | l[1]);
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
  v = swap_max_u64<true>(v);
  v = swap_max_u64<false>(v);
  v = max(v, dpp_u64<0x128>(v));
  v = max(v, dpp_u64<0x124>(v));
  v = max(v, dpp_u64<0x122>(v));
  return max(v, dpp_u64<0x121>(v));
}

// Inclusive sums over the wave by DPP moves (no LDS crossbar): shifts by 1, 2,
// 4 and 8 lanes inside each 16-lane row, then lane 15 of a row into the next
// row (rows 1 and 3) and lane 31 into the upper half.  F adds the value that
// a move brings (0 where the lane has no source).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_zero(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_zero(uint64_t v) {
  return ((uint64_t)dpp_zero<CTRL, ROWS>((uint32_t)(v >> 32)) << 32) | dpp_zero<CTRL, ROWS>((uint32_t)v);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ U128 dpp_zero(U128 v) {
  return U128{dpp_zero<CTRL, ROWS>(v.lo), dpp_zero<CTRL, ROWS>(v.hi)};
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_zero(double v) {
  return __longlong_as_double((long long)dpp_zero<CTRL, ROWS>((uint64_t)__double_as_longlong(v)));
}
__device__ __forceinline__ uint32_t plus(uint32_t a, uint32_t b) { return a + b; }
__device__ __forceinline__ double plus(double a, double b) { return a + b; }
__device__ __forceinline__ U128 plus(U128 a, U128 b) { return u128_add(a, b); }
template <class T>
__device__ __forceinline__ T wave_inscan(T v) {
  v = plus(v, dpp_zero<0x111, 0xF>(v));  // row_shr:1
  v = plus(v, dpp_zero<0x112, 0xF>(v));  // row_shr:2
  v = plus(v, dpp_zero<0x114, 0xF>(v));  // row_shr:4
  v = plus(v, dpp_zero<0x118, 0xF>(v));  // row_shr:8
  v = plus(v, dpp_zero<0x142, 0xA>(v));  // row_bcast:15
  return plus(v, dpp_zero<0x143, 0xC>(v));  // row_bcast:31
}
__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, int lane) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

constexpr int kLevels = 4;  // windows a block considers (level_window)
struct Window {
  int32_t lo, hi;
  uint32_t elements;
};

struct SampleShared {
  union {
    uint32_t hf[kBuckets + 64];  // element counts of the buckets, 64 per-lane spill slots
    struct {
      uint64_t key[kMaxCand];  // (~orderable key) << 32 | position: ascending = nucleus order
      uint64_t e[kMaxCand];    // weights
      uint64_t sa[kMaxSub];    // exact sub-bucket masses of the window
      uint64_t sb[kMaxSub];
      uint32_t scnt[kMaxSub];
    } c;
    struct {
      uint64_t a[kCoarse + 64];  // exact group masses, 64 per-lane spill slots
      uint64_t b[kCoarse + 64];
      uint32_t cnt[256];  // element counts of the key passes
    } h;
  } u;
  uint64_t seg_a[kMaxSeg];  // nucleus mass per segment
  uint64_t seg_b[kMaxSeg];
  uint32_t seg_t[kMaxSeg];  // elements tied at the threshold key per segment
  uint64_t wkey[64];        // the crossing sub-bucket's elements
  uint64_t we[64];
  double tab[kTab];
  float gmass[64];          // estimated masses and element counts of the 64 bucket groups
  uint32_t gcnt[64];
  U128 xred[kSWaves], yred[kSWaves];
  uint64_t kred[kSWaves];
  uint32_t ured[kSWaves];
  uint32_t off[64];
  Window win[kLevels];
  U128 above, claim_base;
  uint32_t tie_base, T;
  int32_t bsel, ncand, cut_idx, cut_pos, claim_seg, tie_seg;
};

__device__ unsigned long long block_max_u64(unsigned long long v, SampleShared& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_max_u64(v);
  __syncthreads();
  if (lane == 0) sh.kred[wave] = v;
  __syncthreads();
  unsigned long long r = sh.kred[0];
  for (int w = 1; w < kSWaves; ++w) r = max(r, (unsigned long long)sh.kred[w]);
  return r;
}

// Exclusive prefix sums over threads (thread order); *total = sum.
__device__ U128 block_exscan_u128(U128 v, SampleShared& sh, U128* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const U128 inc = wave_inscan(v);
  __syncthreads();
  if (lane == 63) sh.xred[wave] = inc;
  __syncthreads();
  U128 base{0ull, 0ull}, tot{0ull, 0ull};
  for (int w = 0; w < kSWaves; ++w) {
    if (w < wave) base = u128_add(base, sh.xred[w]);
    tot = u128_add(tot, sh.xred[w]);
  }
  *total = tot;
  return u128_add(base, u128_sub(inc, v));
}

// Sums of two values over the block, in every thread.
__device__ __forceinline__ void block_sum2_u128(U128 v, U128 w, SampleShared& sh, U128& sv, U128& sw) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const U128 iv = wave_inscan(v), iw = wave_inscan(w);
  __syncthreads();
  if (lane == 63) {
    sh.xred[wave] = iv;
    sh.yred[wave] = iw;
  }
  __syncthreads();
  sv = sh.xred[0];
  sw = sh.yred[0];
  for (int i = 1; i < kSWaves; ++i) {
    sv = u128_add(sv, sh.xred[i]);
    sw = u128_add(sw, sh.yred[i]);
  }
}

__device__ uint32_t block_exscan_u32(uint32_t v, SampleShared& sh, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t inc = wave_inscan(v);
  __syncthreads();
  if (lane == 63) sh.ured[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int w = 0; w < kSWaves; ++w) {
    if (w < wave) base += sh.ured[w];
    tot += sh.ured[w];
  }
  *total = tot;
  return base + inc - v;
}

__device__ __forceinline__ U128 block_sum_u128(U128 v, SampleShared& sh) {
  U128 tot;
  block_exscan_u128(v, sh, &tot);
  return tot;
}

// The lane's four positions p .. p+3; positions past the row are not read and
// give -inf, whose weight is 0 and whose bucket is the last.
__device__ __forceinline__ void load4(const float* __restrict__ row, int n, int p, float (&x)[4]) {
  if (p + 3 < n) {
    float4 q;
    __builtin_memcpy(&q, row + p, 16);  // one load at any alignment
    x[0] = q.x;
    x[1] = q.y;
    x[2] = q.z;
    x[3] = q.w;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = p + e < n ? row[p + e] : -__builtin_inff();
  }
}

// fn(q, p, x) on chunks q0, q0 + step, ... below q1, UN chunks loaded ahead.
template <int UN, class F>
__device__ __forceinline__ void walk_chunks(const float* __restrict__ row, int n, int q0, int q1, int step, F&& fn) {
  const int lane = threadIdx.x & 63;
  for (int q = q0; q < q1; q += UN * step) {
    float x[UN][4];
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (u == 0 || q + u * step < q1) load4(row, n, (q + u * step) * kChunk + 4 * lane, x[u]);
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (u == 0 || q + u * step < q1) fn(q + u * step, (q + u * step) * kChunk + 4 * lane, x[u]);
  }
}

// Every chunk of the row, dealt to the waves in turn.
template <int UN = 2, class F>
__device__ __forceinline__ void for_chunks(const float* __restrict__ row, int n, int NC, F&& fn) {
  walk_chunks<UN>(row, n, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), NC, kSWaves, fn);
}

// Every chunk of the row, each wave on one contiguous range (so that a
// segment's chunks mostly fall to one wave).
template <int UN = 2, class F>
__device__ __forceinline__ void for_chunks_contig(const float* __restrict__ row, int n, int NC, F&& fn) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int per = (NC + kSWaves - 1) / kSWaves;
  walk_chunks<UN>(row, n, wave * per, min(NC, (wave + 1) * per), 1, fn);
}

// ---------------------------------------------------------------------------
// Few rows: the passes over a row are spread over several blocks (launch_sample
// chooses), with the rest of the selection in one block per row as ever.
//   k_sample_count  pass 1 over 1/p1 of a row: its bucket counts, and the
//                   counts and estimated masses of its 64 groups of 64 buckets
//   k_sample_mass   the window from those of all parts (a group, then a
//                   bucket), then the exact pass over spp segments of the row
//   k_sample<true>  takes the parts' sums and lists in place of its own passes

constexpr int kCountParts = 8;   // parts of pass 1
constexpr int kMaxParts = 32;    // parts of the exact pass
constexpr int kPartCand = 128;   // window elements a part can list
constexpr int kPartFull = 0x7FFFFFFF;
constexpr int kMassThreads = 256;

struct SplitScratch {
  uint2* coarse;    // [M][p1][64]: a group's count and mass
  uint32_t* count;  // [M][p1][kBuckets]
  int32_t* win;     // [M][2]: window
  uint64_t* part;   // [M][p2][4]: total (a, b), mass below the window (a, b)
  uint32_t* cnt;    // [M][p2]: window elements
  uint64_t* seg;    // [M][kMaxSeg][2]
  uint64_t* list;   // [M][p2][kPartCand][2]: key, weight
  int p1, p2, spp;
};

// Estimated mass of c elements of bucket b: c times the weight of its middle.
constexpr float kBucketStep = kYSpan / kBuckets;
__device__ __forceinline__ float bucket_weight(int b) { return __expf(-kBucketStep * ((float)b + 0.5f)); }
// An element's weight is within a factor exp(+-kBucketStep / 2) of its bucket's
// middle: 2.934e-3 of it, and 2.6e-5 for the float arithmetic (the place of an
// element, exponentials, sums).  The last bucket's elements count as nothing:
// each weighs below kLastWeight.
constexpr double kMassErr = 2.96e-3, kLastWeight = 3.9e-11;

// The window [lo, hi], found by four waves, one for each share f of the error:
// lane g has the estimated mass and the element count of group g (64 buckets),
// bucket(b) gives a bucket's count.  With A the estimated mass up to some bucket and
// Z that of all, A - p Z = (1 - p) A - p (Z - A) decides whether the cut lies past
// it, and is off by at most
//   err(A) = kMassErr ((1 - p) (A - 1) + p (Z - A)) + p n kLastWeight,
// as the row's maximum weighs 1 exactly and is counted so.  [lo, hi] is what
// lies within err, so it holds the cut.  With more than kSureCand elements
// there, none of which weighs much, the errors of the estimate average out, and
// a shorter list is faster (640 rows of 65536 normal logits of sigma / tau 1.5:
// 106 us, 111 with the whole of err): a quarter of err, a sixteenth if those are
// more than `cap`, else the estimate's bucket alone.  A window that misses the
// cut costs a further exact pass in the row's block, and one such row the whole
// launch.  (us of the sampler with the estimate's bucket, widened within 1e-4 Z
// of its edges, an error that a few large weights exceed / now: 640 x 65536, one
// id of 0.8 of the mass and a normal tail, top_p 0.8, 228 / 103; sigma / tau 4,
// top_p 0.9, 181 / 94; 64 x 65536 of it 112 / 36; 128 x 150000 339 / 71.)
constexpr uint32_t kSureCand = 64;

// The window of one share (level 0 ... 3: f = 1, 1/4, 1/16, 0) of the error, by a wave.
template <class B>
__device__ __forceinline__ Window level_window(double p, int n, int level, double mass, uint32_t count, B&& bucket) {
  const int lane = threadIdx.x & 63;
  auto of_lane = [](double v, int l) {
    return __longlong_as_double((long long)readlane_u64((uint64_t)__double_as_longlong(v), l));
  };
  if (lane == 0) mass += 1.0 - (double)bucket_weight(0);
  const double inc = wave_inscan(mass);
  const uint32_t kinc = wave_inscan(count);
  const double Z = of_lane(inc, 63), need = p * Z, last = p * (double)n * kLastWeight;
  auto err = [&](double A) { return kMassErr * ((1.0 - p) * fmax(A - 1.0, 0.0) + p * (Z - A)) + last; };
  // buckets of the group looked at last: counts up to and in a lane's, masses up to it
  int cg = -1;
  uint32_t ck = 0u, cb = 0u;
  double cA = 0.0;
  // the first bucket whose A reaches `need` with f err(A) added, and the elements
  // before it and up to it (bucket kBuckets: none does)
  auto first = [&](double f, uint32_t& before, uint32_t& upto) {
    const uint64_t hit = __ballot(inc + f * err(inc) >= need);
    if (!hit) {
      before = upto = (uint32_t)n;
      return kBuckets;
    }
    const int g = __ffsll((unsigned long long)hit) - 1;
    if (g != cg) {
      cg = g;
      const uint32_t k = bucket(64 * g + lane);
      double d = (double)((float)k * bucket_weight(64 * g + lane));
      if (g == 0 && lane == 0) d += 1.0 - (double)bucket_weight(0);
      cA = of_lane(inc - mass, g) + wave_inscan(d);
      ck = (uint32_t)__builtin_amdgcn_readlane((int)(kinc - count), g) + wave_inscan(k);
      cb = ck - k;
    }
    const uint64_t hit2 = __ballot(cA + f * err(cA) >= need);
    const int l = hit2 ? __ffsll((unsigned long long)hit2) - 1 : 63;  // (63: rounding of the group's sum)
    before = (uint32_t)__builtin_amdgcn_readlane((int)cb, l);
    upto = (uint32_t)__builtin_amdgcn_readlane((int)ck, l);
    return 64 * g + l;
  };
  const double f = level == 0 ? 1.0 : level == 1 ? 0.25 : level == 2 ? 0.0625 : 0.0;
  uint32_t b0, b1, other;
  Window w;
  w.lo = min(first(f, b0, other), kBuckets - 1);
  w.hi = w.lo;
  w.elements = 0u;  // (the estimate's bucket alone: whatever it holds)
  if (level < kLevels - 1) {
    w.hi = first(-f, other, b1);
    w.elements = b1 - b0;
    w.hi = min(w.hi, kBuckets - 1);
  }
  return w;
}

// The first level with few enough elements.
__device__ __forceinline__ void pick_window(const Window (&w)[kLevels], uint32_t cap, int& lo, int& hi) {
  int k = kLevels - 1;
#pragma unroll
  for (int i = kLevels - 2; i >= 0; --i)
    if (w[i].elements <= (i == 0 ? kSureCand : cap)) k = i;
  lo = w[k].lo;
  hi = w[k].hi;
}

template <int NT>
__device__ __forceinline__ float row_max(const unsigned long long* __restrict__ keys, int nblk,
                                         uint64_t (&red)[NT / 64]) {
  uint64_t k = 0ull;
  for (int i = threadIdx.x; i < nblk; i += NT) k = max(k, (uint64_t)keys[i]);
  k = wave_max_u64(k);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = k;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) k = max(k, red[w]);
  return from_orderable((uint32_t)(k >> 32));
}

// Counts c of thread t's kBPT buckets; count k and estimated mass d of its group
// (valid in every eighth thread).
__device__ __forceinline__ void group_sums(const uint32_t* hf, uint32_t (&c)[kBPT], float& d, uint32_t& k) {
  static_assert(kBPT * 8 == 64, "eight threads per group");
  const int b0 = kBPT * threadIdx.x;
  d = 0.0f;
  k = 0u;
#pragma unroll
  for (int i = 0; i < kBPT; ++i) {
    c[i] = hf[b0 + i];
    k += c[i];
    d += (float)c[i] * bucket_weight(b0 + i);
  }
#pragma unroll
  for (int o = 1; o < 8; o *= 2) {
    k += __shfl_xor(k, o, 64);
    d += __shfl_xor(d, o, 64);
  }
}

__global__ __launch_bounds__(kSThreads) void k_sample_count(const float* __restrict__ f, int n,
                                                            const unsigned long long* __restrict__ best,
                                                            int nblk, float temperature, SplitScratch sc) {
  __shared__ uint32_t hf[kBuckets + 64];
  __shared__ uint64_t red[kSWaves];
  const int m = blockIdx.y, part = blockIdx.x, t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const float* row = f + (int64_t)m * n;
  for (int b = t; b < kBuckets + 64; b += kSThreads) hf[b] = 0u;
  const float vmax = row_max<kSThreads>(best + (int64_t)m * kMaxBlocks, nblk, red);  // and the zeros
  const float kb = (float)kBuckets / (kYSpan * temperature);
  const int NC = (n + kChunk - 1) / kChunk;
  const int q0 = (int)((int64_t)NC * part / sc.p1), q1 = (int)((int64_t)NC * (part + 1) / sc.p1);
  walk_chunks<4>(row, n, q0 + wave, q1, kSWaves, [&](int, int, const float (&x)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      int b = bucket_of(ypos(x[e], vmax, kb));
      if (b == kBuckets - 1) b = kBuckets + lane;
      atomicAdd(&hf[b], 1u);
    }
  });
  __syncthreads();
  const int64_t at = (int64_t)m * sc.p1 + part;
  float d;
  uint32_t k, c[kBPT];
  group_sums(hf, c, d, k);
#pragma unroll
  for (int i = 0; i < kBPT; i += 4)
    *reinterpret_cast<uint4*>(sc.count + at * kBuckets + kBPT * t + i) = make_uint4(c[i], c[i + 1], c[i + 2], c[i + 3]);
  if ((t & 7) == 0) sc.coarse[at * 64 + (t >> 3)] = make_uint2(k, __float_as_uint(d));
}

__global__ __launch_bounds__(kMassThreads) void k_sample_mass(const float* __restrict__ f, int n,
                                                              const unsigned long long* __restrict__ best,
                                                              int nblk, float temperature, float top_p,
                                                              SplitScratch sc) {
  constexpr int NWV = kMassThreads / 64;
  __shared__ double tab[kTab];
  __shared__ uint64_t red[NWV];
  __shared__ uint64_t sums[NWV][4];
  __shared__ Window s_win[kLevels];
  __shared__ uint32_t s_cnt;
  const int m = blockIdx.y, part = blockIdx.x, t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const float* row = f + (int64_t)m * n;
  const int G = kChunk * max(kSegChunks, (n + kChunk * kMaxSeg - 1) / (kChunk * kMaxSeg));
  const int NS = (n + G - 1) / G;
  static_assert(kTab == kMassThreads, "one entry per thread");
  tab[t] = exp2((double)t * (1.0 / kTab));
  if (t == 0) s_cnt = 0u;
  int lo = kBuckets, hi = kBuckets - 1;  // top_p 1: every bucket below lo, no window
  static_assert(NWV == kLevels, "a wave per level");
  if (top_p < 1.0f) {
    // (the parts' values are all loaded before the first is used)
    uint2 cg[kCountParts];
#pragma unroll
    for (int i = 0; i < kCountParts; ++i)
      cg[i] = sc.coarse[((int64_t)m * sc.p1 + min(i, sc.p1 - 1)) * 64 + lane];
    double mass = 0.0;
    uint32_t count = 0u;
#pragma unroll
    for (int i = 0; i < kCountParts; ++i) {
      mass += i < sc.p1 ? (double)__uint_as_float(cg[i].y) : 0.0;
      count += i < sc.p1 ? cg[i].x : 0u;
    }
    auto bucket = [&](int b) {
      uint32_t c[kCountParts], k = 0u;
#pragma unroll
      for (int i = 0; i < kCountParts; ++i) c[i] = sc.count[((int64_t)m * sc.p1 + min(i, sc.p1 - 1)) * kBuckets + b];
#pragma unroll
      for (int i = 0; i < kCountParts; ++i) k += i < sc.p1 ? c[i] : 0u;
      return k;
    };
    const Window w = level_window((double)top_p, n, wave, mass, count, bucket);
    if (lane == 0) s_win[wave] = w;
  }
  const float vmax = row_max<kMassThreads>(best + (int64_t)m * kMaxBlocks, nblk, red);  // and the table, the levels
  // (parts have room for twice their share)
  if (top_p < 1.0f) pick_window(s_win, (uint32_t)min(kMaxCand, kPartCand / 2 * sc.p2), lo, hi);
  if (part == 0 && t == 0) {
    sc.win[2 * m] = lo;
    sc.win[2 * m + 1] = hi;
  }
  const double kk = (double)kTab / (kLn2 * (double)temperature);
  const double c0 = -(double)vmax * kk;
  const float kb = (float)kBuckets / (kYSpan * temperature);
  const float ylo = (float)lo, yhi = (float)(hi + 1);
  const bool window = lo <= hi, last = hi >= kBuckets - 1;
  const int64_t at = (int64_t)m * sc.p2 + part;
  uint64_t* list = sc.list + at * kPartCand * 2;
  uint64_t za = 0ull, zb = 0ull, ma = 0ull, mb = 0ull;
  const int s1 = min(NS, (part + 1) * sc.spp);
  for (int sg = part * sc.spp + wave; sg < s1; sg += NWV) {
    uint64_t sz = 0ull, sm = 0ull;  // at most 128 weights a lane
    walk_chunks<4>(row, n, sg * (G / kChunk), min((sg + 1) * (G / kChunk), (n + kChunk - 1) / kChunk), 1,
                   [&](int, int p, const float (&x)[4]) {
      uint64_t w[4];
      bool cand[4], anyc = false;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        w[e] = weight56(x[e], kk, c0, tab);
        const float y = ypos(x[e], vmax, kb);
        const bool mem = y < ylo || !window;
        sz += w[e];
        sm += mem ? w[e] : 0ull;
        cand[e] = !mem && (last || y < yhi);
        anyc |= cand[e];
      }
      if (__ballot(anyc)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (cand[e] && p + e < n) {
            const uint32_t slot = atomicAdd(&s_cnt, 1u);
            if (slot < (uint32_t)kPartCand) {
              list[2 * slot] = ((uint64_t)(~orderable(x[e])) << 32) | (uint32_t)(p + e);
              list[2 * slot + 1] = w[e];
            }
          }
        }
      }
    });
    za += part_a(sz);
    zb += part_b(sz);
    ma += part_a(sm);
    mb += part_b(sm);
    const uint64_t A = wave_sum_u64(part_a(sm)), B = wave_sum_u64(part_b(sm));
    if (lane == 0) {
      sc.seg[((int64_t)m * kMaxSeg + sg) * 2] = A;
      sc.seg[((int64_t)m * kMaxSeg + sg) * 2 + 1] = B;
    }
  }
  za = wave_sum_u64(za);
  zb = wave_sum_u64(zb);
  ma = wave_sum_u64(ma);
  mb = wave_sum_u64(mb);
  if (lane == 0) {
    sums[wave][0] = za;
    sums[wave][1] = zb;
    sums[wave][2] = ma;
    sums[wave][3] = mb;
  }
  __syncthreads();
  if (t < 4) {
    uint64_t v = 0ull;
#pragma unroll
    for (int w = 0; w < NWV; ++w) v += sums[w][t];
    sc.part[at * 4 + t] = v;
  }
  if (t == 0) sc.cnt[at] = s_cnt;
}

// SPLIT: the passes of the first window were made by the kernels above.
template <bool SPLIT>
__global__ __launch_bounds__(kSThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_sample(
    const float* __restrict__ f, int n, const unsigned long long* __restrict__ best, int nblk,
    const int32_t* __restrict__ ids, int R, float temperature, float top_p, uint32_t seed_lo,
    uint32_t seed_hi, int32_t* __restrict__ tokens, const SplitScratch sc) {
  __shared__ SampleShared sh;
  const int m = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const float* row = f + (int64_t)m * n;
  // segments of G positions (a multiple of the chunk, at least kSegChunks
  // chunks), at most kMaxSeg of them
  const int G = kChunk * max(kSegChunks, (n + kChunk * kMaxSeg - 1) / (kChunk * kMaxSeg));
  const int NS = (n + G - 1) / G;
  const int NC = (n + kChunk - 1) / kChunk;

  if (t < kTab) sh.tab[t] = exp2((double)t * (1.0 / kTab));
  sh.seg_a[t] = 0ull;
  sh.seg_b[t] = 0ull;
  sh.seg_t[t] = 0u;
  if (t == 0) {
    sh.bsel = -1;
    sh.ncand = 0;
    sh.cut_idx = -1;
    sh.cut_pos = n;
    sh.claim_seg = -1;
    sh.tie_seg = -1;
    sh.T = 0u;
  }
  // row maximum from the projection's per-tile argmax keys
  unsigned long long kmax = 0ull;
  for (int i = t; i < nblk; i += kSThreads) kmax = max(kmax, best[(int64_t)m * kMaxBlocks + i]);
  kmax = block_max_u64(kmax, sh);  // its barriers also publish the table and the zeroed state
  const float vmax = from_orderable((uint32_t)(kmax >> 32));
  const double kk = (double)kTab / (kLn2 * (double)temperature);
  const double c0 = -(double)vmax * kk;
  const float kb = (float)kBuckets / (kYSpan * temperature);
  const double* tab = sh.tab;
  auto fix = [&](float x) { return weight56(x, kk, c0, tab); };
  auto member = [&](float x, int pos, uint32_t T, int cut) {
    const uint32_t k = orderable(x);
    return k > T || (k == T && pos <= cut);
  };

  // Exact pass with the window [lo, hi]: segment masses of the buckets below
  // lo, the window's elements into the list.  Returns the total mass Z and the
  // mass `above` of the buckets below lo.  A wave's chunks are contiguous, so
  // each lane sums its share of a segment and the wave reduces it once per
  // segment (one wave-wide sum per chunk cost a quarter of the pass); one vote
  // per chunk skips the list code where no element of the chunk falls in the
  // window.
  auto collect = [&](int lo, int hi, U128& Z, U128& above) {
    uint64_t za = 0ull, zb = 0ull, ma = 0ull, mb = 0ull;
    // the lane's masses in segment cur (at most 128 weights): all, below the window
    uint64_t sz = 0ull, sm = 0ull;
    int cur = -1;
    // floor(y) < b is y < b; the last bucket has no upper end
    const float ylo = (float)lo, yhi = (float)(hi + 1);
    const bool window = lo <= hi, last = hi >= kBuckets - 1;
    auto flush = [&]() {
      za += part_a(sz);
      zb += part_b(sz);
      ma += part_a(sm);
      mb += part_b(sm);
      const uint64_t A = wave_sum_u64(part_a(sm)), B = wave_sum_u64(part_b(sm));
      if (lane == 0 && (A | B)) {
        atomicAdd(reinterpret_cast<unsigned long long*>(&sh.seg_a[cur]), (unsigned long long)A);
        atomicAdd(reinterpret_cast<unsigned long long*>(&sh.seg_b[cur]), (unsigned long long)B);
      }
      sz = 0ull;
      sm = 0ull;
    };
    for_chunks_contig(row, n, NC, [&](int q, int p, const float (&x)[4]) {
      const int sg = q * kChunk / G;
      if (sg != cur) {
        if (cur >= 0) flush();
        cur = sg;
      }
      uint64_t w[4];
      bool cand[4];
      bool anyc = false;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        w[e] = fix(x[e]);
        const float y = ypos(x[e], vmax, kb);
        const bool mem = y < ylo || !window;
        sz += w[e];
        sm += mem ? w[e] : 0ull;
        cand[e] = !mem && (last || y < yhi);
        anyc |= cand[e];
      }
      if (__ballot(anyc)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          cand[e] = cand[e] && p + e < n;
          const uint64_t bal = __ballot(cand[e]);
          if (bal) {
            const int leader = __ffsll((unsigned long long)bal) - 1;
            int base = 0;
            if (lane == leader) base = atomicAdd(&sh.ncand, __popcll(bal));
            base = __builtin_amdgcn_readlane(base, leader);
            if (cand[e]) {
              const int slot = base + __popcll(bal & ((1ull << lane) - 1ull));
              if (slot < kMaxCand) {
                sh.u.c.key[slot] = ((uint64_t)(~orderable(x[e])) << 32) | (uint32_t)(p + e);
                sh.u.c.e[slot] = w[e];
              }
            }
          }
        }
      }
    });
    if (cur >= 0) flush();
    // barriers: segments and list complete
    block_sum2_u128(u128_join(za, zb), u128_join(ma, mb), sh, Z, above);
  };
  // The same from the parts that k_sample_mass wrote (kPartFull if a part
  // listed more than it has room for although the list has).
  auto gather = [&](U128& Z, U128& above) {
    const uint64_t* pt = sc.part + (int64_t)m * sc.p2 * 4;
    U128 z{0ull, 0ull}, a{0ull, 0ull};
    uint32_t c = 0u;
    if (t < sc.p2) {
      z = u128_join(pt[4 * t], pt[4 * t + 1]);
      a = u128_join(pt[4 * t + 2], pt[4 * t + 3]);
      c = sc.cnt[(int64_t)m * sc.p2 + t];
    }
    if (t < NS) {
      sh.seg_a[t] = sc.seg[((int64_t)m * kMaxSeg + t) * 2];
      sh.seg_b[t] = sc.seg[((int64_t)m * kMaxSeg + t) * 2 + 1];
    }
    if (wave == 0) {
      static_assert(kMaxParts < 64, "a wave scans the parts");
      const uint32_t inc = wave_inscan(c);
      const bool fits = __ballot(c > (uint32_t)kPartCand) == 0ull;
      if (lane <= sc.p2) sh.off[lane] = inc - c;  // (lane p2: the total)
      if (lane == 0) {
        const int nc = __builtin_amdgcn_readlane((int)inc, 63);
        sh.ncand = fits || nc > kMaxCand ? nc : kPartFull;
      }
    }
    block_sum2_u128(z, a, sh, Z, above);  // (and its barriers)
    if (sh.ncand <= kMaxCand) {
      for (int i = t; i < sc.p2 * kPartCand; i += kSThreads) {
        const int p = i / kPartCand, e = i % kPartCand;
        const uint32_t o = sh.off[p] + e;
        if (o < sh.off[p + 1]) {
          const uint64_t* src = sc.list + ((int64_t)m * sc.p2 * kPartCand + i) * 2;
          sh.u.c.key[o] = src[0];
          sh.u.c.e[o] = src[1];
        }
      }
    }
    __syncthreads();
  };
  const bool all = !(top_p < 1.0f);
  int lo = kBuckets, hi = kBuckets - 1;  // all: every bucket below lo, no window
  if constexpr (SPLIT) {
    lo = sc.win[2 * m];
    hi = sc.win[2 * m + 1];
  } else if (!all) {
    // 1. histogram of element counts -> window
    for (int b = t; b < kBuckets + 64; b += kSThreads) sh.u.hf[b] = 0u;
    __syncthreads();
    for_chunks(row, n, NC, [&](int, int p, const float (&x)[4]) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float y = ypos(x[e], vmax, kb);
        // the last bucket, which many may share (positions past the row among
        // them), counts in a slot per lane: its weight is nil
        int b = bucket_of(y);
        if (b == kBuckets - 1) b = kBuckets + lane;
        atomicAdd(&sh.u.hf[b], 1u);
      }
    });
    __syncthreads();
    float d;
    uint32_t k, c[kBPT];
    group_sums(sh.u.hf, c, d, k);
    if ((t & 7) == 0) {
      sh.gmass[t >> 3] = d;
      sh.gcnt[t >> 3] = k;
    }
    __syncthreads();
    if (wave < kLevels) {
      const Window w = level_window((double)top_p, n, __builtin_amdgcn_readfirstlane(wave), (double)sh.gmass[lane],
                                    sh.gcnt[lane], [&](int b) { return sh.u.hf[b]; });
      if (lane == 0) sh.win[wave] = w;
    }
    __syncthreads();  // (and the list may take the histogram's place)
    pick_window(sh.win, (uint32_t)kMaxCand, lo, hi);
  }

  // 2. exact pass: Z, segment masses below the window, the window's list; then
  // the list's sub-bucket that holds the cut.  A narrowed window may have missed
  // the cut, or overflow the list: the pass is redone on another window next to
  // it, three times at most, then on the group of 4 buckets that an exact
  // histogram gives.
  U128 need{0ull, 0ull}, above;
  int nc = 0, nsub = 0, wsh = 0, ss = -1;
  auto sub_of = [&](uint64_t key) {
    const float x = from_orderable(~(uint32_t)(key >> 32));
    return min(max(subbucket_of(ypos(x, vmax, kb)) - kSub * lo, 0) >> wsh, nsub - 1);
  };
  bool group = false;  // [lo, hi] holds the cut
  for (int tries = 0;; ++tries) {
    U128 Z;
    if (SPLIT && tries == 0) gather(Z, above);
    else collect(lo, hi, Z, above);
    if (all) break;
    if (tries == 0) {
      need = u128_ceil((double)top_p * u128_to_f64(Z));
      if (need.lo == 0ull && need.hi == 0ull) need.lo = 1ull;
    }
    nc = sh.ncand;
    const bool below = !u128_lt(above, need), over = nc > kMaxCand;
    if (!below && !over) {
      // exact histogram of the list over sub-buckets of the window
      wsh = hi - lo < 4 ? 0 : 30 - __clz(hi - lo);  // so that kSub (hi - lo + 1) >> wsh <= kMaxSub
      nsub = min(kMaxSub, kSub * (hi - lo + 1));
      sh.u.c.sa[t] = 0ull;
      sh.u.c.sb[t] = 0ull;
      sh.u.c.scnt[t] = 0u;
      if (t == 0) sh.bsel = -1;
      __syncthreads();
      for (int i = t; i < nc; i += kSThreads) {
        const int s = sub_of(sh.u.c.key[i]);
        const uint64_t w = sh.u.c.e[i];
        atomicAdd(reinterpret_cast<unsigned long long*>(&sh.u.c.sa[s]), (unsigned long long)part_a(w));
        atomicAdd(reinterpret_cast<unsigned long long*>(&sh.u.c.sb[s]), (unsigned long long)part_b(w));
        atomicAdd(&sh.u.c.scnt[s], 1u);
      }
      __syncthreads();
      const U128 st = u128_join(sh.u.c.sa[t], sh.u.c.sb[t]);
      U128 tot;
      const U128 sx = u128_add(above, block_exscan_u128(st, sh, &tot));
      if (t < nsub && u128_lt(sx, need) && !u128_lt(u128_add(sx, st), need)) {
        sh.bsel = t;
        sh.above = sx;
      }
      __syncthreads();
      ss = sh.bsel;  // -1: the cut lies past the window
      if (ss >= 0) break;
    }
    if (group) break;
    __syncthreads();
    if (SPLIT && nc == kPartFull && !below) {
      // the same window in this block
    } else if (tries < 3 && below && lo > 0) {
      hi = lo - 1;
      lo = max(0, lo - 2);
    } else if (tries < 3 && !below && over && hi > lo) {
      --hi;
    } else if (tries < 3 && !below && !over && hi < kBuckets - 1) {
      lo = hi + 1;
      hi = min(hi + 2, kBuckets - 1);
    } else {
      group = true;
      for (int b = t; b < kCoarse + 64; b += kSThreads) {
        sh.u.h.a[b] = 0ull;
        sh.u.h.b[b] = 0ull;
      }
      if (t == 0) sh.bsel = -1;
      __syncthreads();
      for_chunks(row, n, NC, [&](int, int p, const float (&x)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint64_t w = fix(x[e]);
          int b = bucket_of(ypos(x[e], vmax, kb)) >> 2;
          if (b == kCoarse - 1) b = kCoarse + lane;
          atomicAdd(reinterpret_cast<unsigned long long*>(&sh.u.h.a[b]), (unsigned long long)part_a(w));
          atomicAdd(reinterpret_cast<unsigned long long*>(&sh.u.h.b[b]), (unsigned long long)part_b(w));
        }
      });
      __syncthreads();
      if (wave == 0) {
        const uint64_t ta = wave_sum_u64(sh.u.h.a[kCoarse + lane]);
        const uint64_t tb = wave_sum_u64(sh.u.h.b[kCoarse + lane]);
        if (lane == 0) {
          sh.u.h.a[kCoarse - 1] += ta;
          sh.u.h.b[kCoarse - 1] += tb;
        }
      }
      __syncthreads();
      const U128 s0 = u128_join(sh.u.h.a[2 * t], sh.u.h.b[2 * t]);
      const U128 s1 = u128_join(sh.u.h.a[2 * t + 1], sh.u.h.b[2 * t + 1]);
      U128 tot;
      const U128 x0 = block_exscan_u128(u128_add(s0, s1), sh, &tot);
      const U128 x1 = u128_add(x0, s0);
      if (u128_lt(x0, need) && !u128_lt(x1, need)) sh.bsel = 2 * t;
      if (u128_lt(x1, need) && !u128_lt(u128_add(x1, s1), need)) sh.bsel = 2 * t + 1;
      __syncthreads();
      const int cg = max(sh.bsel, 0);
      lo = 4 * cg;
      hi = 4 * cg + 3;
    }
    if (t == 0) sh.ncand = 0;
    sh.seg_a[t] = 0ull;
    sh.seg_b[t] = 0ull;
    __syncthreads();
  }
  if (!all) {
    if (nc <= kMaxCand) {
      ss = max(ss, 0);
      const U128 as = sh.above;
      const uint32_t cs = sh.u.c.scnt[ss];
      if (cs <= 64u) {
        if (wave == 0) {
          // gather sub-bucket ss, then rank it by (key desc, position asc)
          int got = 0;
          for (int base = 0; base < nc; base += 64) {
            const int i = base + lane;
            const bool in = i < nc && sub_of(sh.u.c.key[i]) == ss;
            const uint64_t bal = __ballot(in);
            if (in) {
              const int slot = got + __popcll(bal & ((1ull << lane) - 1ull));
              sh.wkey[slot] = sh.u.c.key[i];
              sh.we[slot] = sh.u.c.e[i];
            }
            got += __popcll(bal);
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
          if (lane < got) {
            const uint64_t kj = sh.wkey[lane];
            uint64_t A = 0ull;  // at most 64 weights
            for (int i = 0; i < got; ++i) A += sh.wkey[i] < kj ? sh.we[i] : 0ull;
            const U128 ex = u128_add(as, U128{A, 0ull});
            const U128 in = u128_add(ex, U128{sh.we[lane], 0ull});
            if (u128_lt(ex, need) && !u128_lt(in, need)) {
              sh.T = ~(uint32_t)(kj >> 32);
              sh.cut_pos = (int)(uint32_t)kj;
            }
          }
        }
        __syncthreads();
        // members of the window: sub-buckets before ss, and ss up to the cut
        const uint64_t kc = ((uint64_t)(~sh.T) << 32) | (uint32_t)sh.cut_pos;
        for (int i = t; i < nc; i += kSThreads) {
          const uint64_t key = sh.u.c.key[i];
          const int s = sub_of(key);
          if (s < ss || (s == ss && key <= kc)) {
            const int pos = (int)(uint32_t)key;
            atomicAdd(reinterpret_cast<unsigned long long*>(&sh.seg_a[pos / G]),
                      (unsigned long long)part_a(sh.u.c.e[i]));
            atomicAdd(reinterpret_cast<unsigned long long*>(&sh.seg_b[pos / G]),
                      (unsigned long long)part_b(sh.u.c.e[i]));
          }
        }
      } else {
        // a crowded sub-bucket: bitonic sort of the list, scan, cut
        int P = 1;
        while (P < nc) P <<= 1;
        for (int i = nc + t; i < P; i += kSThreads) {
          sh.u.c.key[i] = ~0ull;
          sh.u.c.e[i] = 0ull;
        }
        __syncthreads();
        for (int k = 2; k <= P; k <<= 1) {
          for (int j = k >> 1; j > 0; j >>= 1) {
            if (t < P / 2) {
              const int i = 2 * t - (t & (j - 1));
              const int l = i + j;
              const uint64_t ki = sh.u.c.key[i], kl = sh.u.c.key[l];
              if ((ki > kl) == ((i & k) == 0)) {
                sh.u.c.key[i] = kl;
                sh.u.c.key[l] = ki;
                const uint64_t ei = sh.u.c.e[i];
                sh.u.c.e[i] = sh.u.c.e[l];
                sh.u.c.e[l] = ei;
              }
            }
            __syncthreads();
          }
        }
        const int i0 = 2 * t, i1 = 2 * t + 1;
        const U128 e0{i0 < nc ? sh.u.c.e[i0] : 0ull, 0ull};
        const U128 e1{i1 < nc ? sh.u.c.e[i1] : 0ull, 0ull};
        U128 tot2;
        const U128 ex0 = u128_add(above, block_exscan_u128(u128_add(e0, e1), sh, &tot2));
        const U128 ex1 = u128_add(ex0, e0);
        if (i0 < nc && u128_lt(ex0, need) && !u128_lt(ex1, need)) sh.cut_idx = i0;
        if (i1 < nc && u128_lt(ex1, need) && !u128_lt(u128_add(ex1, e1), need)) sh.cut_idx = i1;
        __syncthreads();
        const int jc = sh.cut_idx;
        for (int i = t; i <= jc; i += kSThreads) {
          const int pos = (int)(uint32_t)sh.u.c.key[i];
          atomicAdd(reinterpret_cast<unsigned long long*>(&sh.seg_a[pos / G]),
                    (unsigned long long)part_a(sh.u.c.e[i]));
          atomicAdd(reinterpret_cast<unsigned long long*>(&sh.seg_b[pos / G]),
                    (unsigned long long)part_b(sh.u.c.e[i]));
        }
        if (t == 0 && jc >= 0) {
          sh.T = ~(uint32_t)(sh.u.c.key[jc] >> 32);
          sh.cut_pos = (int)(uint32_t)sh.u.c.key[jc];
        }
      }
    } else {
      // exact radix select, 8 bits per pass, on the keys of the window
      auto in_window = [&](float x) {
        const int b = bucket_of(ypos(x, vmax, kb));
        return b >= lo && b <= hi;
      };
      uint32_t Tk = 0u, kmask = 0u, nt = 0u;
      U128 ab = above;
      for (int shift = 24; shift >= 0; shift -= 8) {
        __syncthreads();  // earlier readers of the histogram are done
        if (t < 256) {
          sh.u.h.a[t] = 0ull;
          sh.u.h.b[t] = 0ull;
          sh.u.h.cnt[t] = 0u;
        }
        if (t == 0) sh.bsel = -1;
        __syncthreads();
        for_chunks(row, n, NC, [&](int, int p, const float (&x)[4]) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t key = orderable(x[e]);
            if (p + e < n && in_window(x[e]) && (key & kmask) == Tk) {
              const int b = (int)((key >> shift) & 255u);
              const uint64_t w = fix(x[e]);
              atomicAdd(reinterpret_cast<unsigned long long*>(&sh.u.h.a[b]), (unsigned long long)part_a(w));
              atomicAdd(reinterpret_cast<unsigned long long*>(&sh.u.h.b[b]), (unsigned long long)part_b(w));
              atomicAdd(&sh.u.h.cnt[b], 1u);
            }
          }
        });
        __syncthreads();
        // thread t < 256 owns key bucket 255 - t: descending keys
        const U128 ks =
            t < 256 ? u128_join(sh.u.h.a[255 - t], sh.u.h.b[255 - t]) : U128{0ull, 0ull};
        U128 ktot;
        const U128 kacc = u128_add(ab, block_exscan_u128(ks, sh, &ktot));
        if (t < 256 && u128_lt(kacc, need) && !u128_lt(u128_add(kacc, ks), need)) {
          sh.bsel = 255 - t;
          sh.above = kacc;
        }
        __syncthreads();
        const int sel = max(sh.bsel, 0);
        ab = sh.bsel >= 0 ? sh.above : ab;
        nt = sh.u.h.cnt[sel];
        Tk |= (uint32_t)sel << shift;
        kmask |= 255u << shift;
      }
      // the c-th element tied at Tk in id order completes the nucleus:
      // smallest c >= 1 with ab + c * E(Tk) >= need
      const U128 WT{fix(from_orderable(Tk)), 0ull};
      const double cd = ceil(u128_to_f64(u128_sub(need, ab)) / u128_to_f64(WT));
      uint32_t c = cd < 1.0 ? 1u : (cd > (double)nt ? nt : (uint32_t)cd);
      while (c > 1u && !u128_lt(u128_add(ab, u128_mul32(WT, c - 1u)), need)) --c;
      while (c < nt && u128_lt(u128_add(ab, u128_mul32(WT, c)), need)) ++c;
      // ties per segment, then the segment and the lane holding the c-th
      for_chunks(row, n, NC, [&](int q, int p, const float (&x)[4]) {
        uint32_t ties = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) ties += (p + e < n && orderable(x[e]) == Tk) ? 1u : 0u;
        ties = (uint32_t)wave_sum_u64(ties);
        if (lane == 0 && ties) atomicAdd(&sh.seg_t[q * kChunk / G], ties);
      });
      __syncthreads();
      const uint32_t tc = t < NS ? sh.seg_t[t] : 0u;
      uint32_t ttot;
      const uint32_t tb = block_exscan_u32(tc, sh, &ttot);
      if (tb < c && c <= tb + tc) {
        sh.tie_seg = t;
        sh.tie_base = tb;
      }
      __syncthreads();
      if (wave == 0 && sh.tie_seg >= 0) {
        const int sg = sh.tie_seg;
        uint32_t run = sh.tie_base;
        const int end = min(n, (sg + 1) * G);
        for (int cb = sg * G; cb < end; cb += kChunk) {
          const int p = cb + 4 * lane;
          float x[4];
          load4(row, n, p, x);
          bool tie[4];
          uint32_t lt = 0u;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            tie[e] = p + e < n && orderable(x[e]) == Tk;
            lt += tie[e] ? 1u : 0u;
          }
          const uint32_t inc = wave_inscan(lt);
          uint32_t seen = run + inc - lt;
          int hit = -1;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (tie[e] && ++seen == c && hit < 0) hit = p + e;
          const uint64_t bal = __ballot(hit >= 0);
          if (bal) {
            const int pos = __shfl(hit, __ffsll((unsigned long long)bal) - 1, 64);
            if (lane == 0) {
              sh.T = Tk;
              sh.cut_pos = pos;
            }
            break;
          }
          run += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        }
      }
      __syncthreads();
      // members of the window
      const uint32_t Tw = sh.T;
      const int cw = sh.cut_pos;
      for_chunks(row, n, NC, [&](int q, int p, const float (&x)[4]) {
        uint64_t A = 0ull, B = 0ull;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (p + e < n && in_window(x[e]) && member(x[e], p + e, Tw, cw)) {
            const uint64_t w = fix(x[e]);
            A += part_a(w);
            B += part_b(w);
          }
        }
        A = wave_sum_u64(A);
        B = wave_sum_u64(B);
        if (lane == 0 && (A | B)) {
          const int sg = q * kChunk / G;
          atomicAdd(reinterpret_cast<unsigned long long*>(&sh.seg_a[sg]), (unsigned long long)A);
          atomicAdd(reinterpret_cast<unsigned long long*>(&sh.seg_b[sg]), (unsigned long long)B);
        }
      });
    }
    __syncthreads();
  }
  // Nucleus: key > T, or key == T and position <= cut (T = 0, cut = n: all).
  const uint32_t T = sh.T;
  const int cut = sh.cut_pos;

  // 3. segment masses in id order, then the inverse CDF inside one segment
  const U128 sm = t < NS ? u128_join(sh.seg_a[t], sh.seg_b[t]) : U128{0ull, 0ull};
  U128 mass;
  const U128 sb = block_exscan_u128(sm, sh, &mass);
  const uint32_t s_idx = (uint32_t)(m / R), r_idx = (uint32_t)(m % R);
  const uint32_t u24 = philox_x0(r_idx, s_idx, 0u, 0u, seed_lo, seed_hi) >> 8;
  const U128 target = u128_mul32(mass, u24);
  if (!u128_lt(target, u128_shl24(sb)) && u128_lt(target, u128_shl24(u128_add(sb, sm)))) {
    sh.claim_seg = t;
    sh.claim_base = sb;
  }
  __syncthreads();
  // the claimed segment in groups of kSegChunks chunks, a wave each: the wave
  // whose chunk holds the target finds the position
  const int sg = sh.claim_seg;
  bool done = false;
  if (sg >= 0) {
    U128 run = sh.claim_base;
    const int end = min(n, (sg + 1) * G);
    for (int cg = sg * G; cg < end && !done; cg += kSegChunks * kChunk) {
      const int p = cg + wave * kChunk + 4 * lane;
      uint64_t li[4];  // the lane's mass up to each of its positions
      U128 inc{0ull, 0ull};
      if (wave < kSegChunks) {
        float x[4];
        load4(row, p < end ? n : 0, p, x);
        uint64_t l = 0ull;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (p + e < end && member(x[e], p + e, T, cut)) l += fix(x[e]);
          li[e] = l;
        }
        inc = wave_inscan(U128{l, 0ull});
        if (lane == 63) sh.xred[wave] = inc;
      }
      __syncthreads();
      U128 before = run;
#pragma unroll
      for (int c = 0; c < kSegChunks; ++c) {
        if (c < wave) before = u128_add(before, sh.xred[c]);
        run = u128_add(run, sh.xred[c]);
      }
      if (wave < kSegChunks && !u128_lt(target, u128_shl24(before)) &&
          u128_lt(target, u128_shl24(u128_add(before, sh.xred[wave])))) {
        const U128 lb = u128_add(before, u128_sub(inc, U128{li[3], 0ull}));
        int hit = -1;
#pragma unroll
        for (int e = 3; e >= 0; --e)
          if (u128_lt(target, u128_shl24(u128_add(lb, U128{li[e], 0ull})))) hit = e;
        const uint64_t bal = __ballot(hit >= 0);
        if (lane == __ffsll((unsigned long long)bal) - 1) tokens[m] = ids[p + hit];
      }
      done = u128_lt(target, u128_shl24(run));
      __syncthreads();  // before the next group's sums
    }
  }
  if (!done && t == 0) tokens[m] = ids[0];
}

__global__ void k_accept(const int32_t* __restrict__ tokens, const int32_t* __restrict__ drafts,
                         int n_sessions, int R, int32_t* __restrict__ accept) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_sessions) return;
  const int kd = R - 1;
  int a = 0;
  bool run = true;
  // tokens and drafts are loaded eight at a time, before any comparison
  for (int b = 0; b < kd && run; b += 8) {
    int32_t t[8], d[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool ok = b + u < kd;
      t[u] = ok ? tokens[(int64_t)s * R + b + u] : 0;
      d[u] = ok ? drafts[(int64_t)s * kd + b + u] : 0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (run && b + u < kd && t[u] == d[u]) ++a;
      else run = false;
    }
  }
  accept[s] = a;
}

// Whether the passes are spread over several blocks: two more launches, for
// rows that keep one block busy longer than that.  Measured (one block / spread,
// tau 0.7, top_p 0.9): 5 rows x 16384 22.0 / 27.5 us, x 32768 32.6 / 27.2,
// x 65536 55.1 / 28.8; 64 rows x 32768 32.6 / 31.0; 128 rows x 32768 33.5 /
// 38.3, x 65536 55.5 / 52.0, x 150000 119 / 77.
static bool split_rows(int64_t M, int64_t n) {
  return M > 0 && M <= 128 && n >= std::max<int64_t>(32768, 512 * M) && n <= 0x7FFFFFFF;
}

struct SplitPlan {
  int p1, p2, spp;
};
static SplitPlan split_plan(int M, int n) {
  const int NC = (n + kChunk - 1) / kChunk;
  const int G = kChunk * std::max(kSegChunks, (n + kChunk * kMaxSeg - 1) / (kChunk * kMaxSeg));
  const int NS = (n + G - 1) / G;
  SplitPlan p;
  p.p1 = std::min(kCountParts, (NC + 31) / 32);
  p.spp = 4 * ((NS + 4 * kMaxParts - 1) / (4 * kMaxParts));
  p.p2 = (NS + p.spp - 1) / p.spp;
  return p;
}

static size_t take(uint8_t* base, size_t& at, size_t bytes, void** out) {
  if (out) *out = base + at;
  at += (bytes + 255) & ~(size_t)255;
  return at;
}

static size_t split_layout(int M, const SplitPlan& p, uint8_t* base, SplitScratch* sc) {
  size_t at = 0;
  void* q[7];
  take(base, at, (size_t)M * p.p1 * 64 * 8, &q[0]);
  take(base, at, (size_t)M * p.p1 * kBuckets * 4, &q[1]);
  take(base, at, (size_t)M * 8, &q[2]);
  take(base, at, (size_t)M * p.p2 * 32, &q[3]);
  take(base, at, (size_t)M * p.p2 * 4, &q[4]);
  take(base, at, (size_t)M * kMaxSeg * 16, &q[5]);
  take(base, at, (size_t)M * p.p2 * kPartCand * 16, &q[6]);
  if (sc)
    *sc = SplitScratch{(uint2*)q[0], (uint32_t*)q[1], (int32_t*)q[2], (uint64_t*)q[3],
                       (uint32_t*)q[4], (uint64_t*)q[5], (uint64_t*)q[6], p.p1, p.p2, p.spp};
  return at;
}

size_t sample_scratch_bytes(int64_t M, int64_t n) {
  if (!split_rows(M, n)) return 0;
  return split_layout((int)M, split_plan((int)M, (int)n), nullptr, nullptr);
}

hipError_t launch_sample(const float* f, int M, int n, const unsigned long long* best, int nblk,
                         const int32_t* ids, int R, float temperature, float top_p, uint64_t seed,
                         int32_t* tokens, void* scratch, hipStream_t s) {
  if (n < 1 || nblk < 1 || nblk > kMaxBlocks) return hipErrorInvalidValue;
  if ((int64_t)(n + kChunk * kMaxSeg - 1) / (kChunk * kMaxSeg) * kChunk * kMaxSeg >= (1ll << 31))
    return hipErrorInvalidValue;
  const uint32_t lo = (uint32_t)seed, hi = (uint32_t)(seed >> 32);
  SplitScratch sc{};
  if (!scratch || !split_rows(M, n)) {
    launch_kernel(k_sample<false>, dim3(M), dim3(kSThreads), 0, s, f, n, best, nblk, ids, R, temperature,
                  top_p, lo, hi, tokens, sc);
    return hipGetLastError();
  }
  const SplitPlan p = split_plan(M, n);
  split_layout(M, p, static_cast<uint8_t*>(scratch), &sc);
  if (top_p < 1.0f)
    launch_kernel(k_sample_count, dim3(p.p1, M), dim3(kSThreads), 0, s, f, n, best, nblk, temperature, sc);
  launch_kernel(k_sample_mass, dim3(p.p2, M), dim3(kMassThreads), 0, s, f, n, best, nblk, temperature, top_p, sc);
  launch_kernel(k_sample<true>, dim3(M), dim3(kSThreads), 0, s, f, n, best, nblk, ids, R, temperature,
                top_p, lo, hi, tokens, sc);
  return hipGetLastError();
}

hipError_t launch_accept(const int32_t* tokens, const int32_t* drafts, int n_sessions, int R,
                         int32_t* accept, hipStream_t s) {
  launch_kernel(k_accept, dim3((n_sessions + 255) / 256), dim3(256), 0, s, tokens, drafts,
                     n_sessions, R, accept);
  return hipGetLastError();
}

}  // namespace sph
