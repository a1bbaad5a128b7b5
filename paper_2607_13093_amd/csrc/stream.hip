// Cloud projection of 9 to 192 rows (MFMA path, HBM bound), and of up to 1024
// over few positions in groups of at most 192 (stream_groups).
//
//   C[m, j] = sum_k h[m, k] * W[S_j, k]      (eq. 12 on the subset S)
//
// With up to 192 rows a launch is a stream over the gathered weight rows: a
// CU's share of the memory rate brings a 32 KB weight stage in about 1.3 us,
// longer than its MFMAs take.  What bounds a two-stage kernel here is the
// latency of the one stage it has in flight (3 TB/s on 14 to 80 rows), so a
// block holds all rows of h (BM = 32 ... 192) and the rest of the LDS goes to
// stages: RW lines of the weights and RA of h, waited for by a counted vmcnt so
// that the younger ones stay in flight across the barrier.  18 rows x 45001 x
// 4000 columns 139 -> 63 us (5.8 TB/s), 18 x 60000 x 3840 96 -> 76, 128 rows
// 92, 155 rows x 4000 182 -> 117 (there the copies of h, 40% of what a CU
// copies at some 28 GB/s, come on top).
//
//  * Every block has an equal share of the positions: a.width of them (at
//    most BN), one round of blocks on the 256 CUs per 65536 positions.  With
//    fixed 256-position tiles 45001 positions left 80 CUs idle and 66096
//    needed a second round for 3 tiles.
//  * A stage is one 128-byte line (narrow blocks: two) of every weight row of the
//    block (64 bf16 or 128 E4M3 columns) and the same columns of h.  The lines are copied
//    global-to-LDS (8 rows per instruction) and non-temporally: 7.3 against
//    6.1 TB/s for plain copies in a probe of this chip; 60000 x 3840 columns
//    18 rows 84 -> 75 us, 90 rows 93 -> 78.  That pays only for whole lines
//    (a line fetched in two parts is fetched twice: 18 x 45001 x 4000 columns
//    87 -> 91), so rows that do not start on a line are still read line by
//    line: stage t holds the row's t-th line and a lane takes its columns from
//    stage t or t + 1, wherever the row's offset puts them (91 -> 63).
//  * Fewer stages of h than of weights where not four of both fit: 155 rows x
//    60000 x 4000 columns 127 -> 117 us, 80 rows 107 -> 93.
//  * 16-byte chunks are XOR-swizzled per row so that fragment reads are
//    conflict-free (rows at different places of their lines meet: 0.65 conflict
//    cycles an LDS instruction on 155 rows x 60000 x 4000).  The reads are inline
//    asm that ends with its own wait: the compiler would make an LDS read wait for
//    every copy in flight.
//  * Every output sums its products in the order of the columns, 16 per MFMA,
//    as the other MFMA kernels do: a row's logits do not depend on the batch.
//  * E4M3 codes are widened to bf16 in registers (exact).
#include <algorithm>

#include "mfma_tile.h"

namespace sph {

typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

constexpr int kStageRow = 128;  // bytes of a weight row per stage

// Waves: one per SIMD up to 64 rows, else two, so that one waits for its
// fragment reads while the other's MFMAs run (128 rows x 60000 x 3840: 104 ->
// 92 us).
constexpr int stream_waves(int bm) { return bm >= 96 ? 8 : 4; }

constexpr int kLdsBytes = 160 * 1024;

// The fragments of NK sub-steps and the wait for them: FM of h at pa[s], 32
// rows (4 KB) apart, and FN of the weights at pb[s][j], 16 bytes a lane (bf16)
// or 8 (E4M3).  One asm block, so that nothing can use or move a register
// before its read has landed.
template <int FM, int FN, int NK, int WT>
struct ReadFrags;
#define SPH_A(s, i, o) "ds_read_b128 %[a" #s #i "], %[p" #s "] offset:" #o "\n"
#define SPH_B(I, s, j) I " %[b" #s #j "], %[q" #s #j "]\n"
#define SPH_AO(s, i) [a##s##i] "=&v"(a[s][i])
#define SPH_BO(s, j) [b##s##j] "=&v"(b[s][j])
#define SPH_TA1(s) SPH_A(s, 0, 0)
#define SPH_TA2(s) SPH_TA1(s) SPH_A(s, 1, 4096)
#define SPH_TA3(s) SPH_TA2(s) SPH_A(s, 2, 8192)
#define SPH_TA4(s) SPH_TA3(s) SPH_A(s, 3, 12288)
#define SPH_TA5(s) SPH_TA4(s) SPH_A(s, 4, 16384)
#define SPH_TB1(I, s) SPH_B(I, s, 0)
#define SPH_TB2(I, s) SPH_TB1(I, s) SPH_B(I, s, 1)
#define SPH_OA1(s) SPH_AO(s, 0)
#define SPH_OA2(s) SPH_OA1(s), SPH_AO(s, 1)
#define SPH_OA3(s) SPH_OA2(s), SPH_AO(s, 2)
#define SPH_OA4(s) SPH_OA3(s), SPH_AO(s, 3)
#define SPH_OA5(s) SPH_OA4(s), SPH_AO(s, 4)
#define SPH_OB1(s) SPH_BO(s, 0)
#define SPH_OB2(s) SPH_OB1(s), SPH_BO(s, 1)
#define SPH_IA(s) [p##s] "v"(pa[s])
#define SPH_IB1(s) [q##s##0] "v"(pb[s][0])
#define SPH_IB2(s) SPH_IB1(s), [q##s##1] "v"(pb[s][1])
#define SPH_T(FM, FN, I, s) SPH_TA##FM(s) SPH_TB##FN(I, s)
#define SPH_OUT(FM, FN, s) SPH_OA##FM(s), SPH_OB##FN(s)
#define SPH_IN(FN, s) SPH_IA(s), SPH_IB##FN(s)
#define SPH_T2(FM, FN, I) SPH_T(FM, FN, I, 0) SPH_T(FM, FN, I, 1)
#define SPH_T4(FM, FN, I) SPH_T2(FM, FN, I) SPH_T(FM, FN, I, 2) SPH_T(FM, FN, I, 3)
#define SPH_OUT2(FM, FN) SPH_OUT(FM, FN, 0), SPH_OUT(FM, FN, 1)
#define SPH_OUT4(FM, FN) SPH_OUT2(FM, FN), SPH_OUT(FM, FN, 2), SPH_OUT(FM, FN, 3)
#define SPH_IN2(FN) SPH_IN(FN, 0), SPH_IN(FN, 1)
#define SPH_IN4(FN) SPH_IN2(FN), SPH_IN(FN, 2), SPH_IN(FN, 3)
#define SPH_READ_FRAGS(FM, FN, NK, WT, I)                                                      \
  template <>                                                                                  \
  struct ReadFrags<FM, FN, NK, WT> {                                                           \
    typedef std::conditional<WT == 0, u32x4_t, u32x2_t>::type B;                               \
    static __device__ __forceinline__ void run(u32x4_t (&a)[NK][FM], B (&b)[NK][FN],           \
                                               const uint32_t (&pa)[NK],                       \
                                               const uint32_t (&pb)[NK][FN]) {                 \
      asm volatile(SPH_T##NK(FM, FN, I) "s_waitcnt lgkmcnt(0)"                                 \
                   : SPH_OUT##NK(FM, FN)                                                       \
                   : SPH_IN##NK(FN)                                                            \
                   : "memory");                                                                \
    }                                                                                          \
  };
#define SPH_READ_BOTH(FM, FN, NK)                      \
  SPH_READ_FRAGS(FM, FN, NK, 0, "ds_read_b128")        \
  SPH_READ_FRAGS(FM, FN, NK, 1, "ds_read_b64")
SPH_READ_BOTH(1, 1, 4)
SPH_READ_BOTH(1, 2, 4)
SPH_READ_BOTH(2, 1, 4)
SPH_READ_BOTH(2, 2, 2)
SPH_READ_BOTH(3, 1, 2)
SPH_READ_BOTH(3, 2, 2)
SPH_READ_BOTH(4, 1, 2)
SPH_READ_BOTH(4, 2, 2)
SPH_READ_BOTH(5, 1, 2)
SPH_READ_BOTH(5, 2, 2)

typedef __attribute__((address_space(3))) const char* lds_cptr_t;

// Clears the 16-byte chunks at and past `valid` of a staged tile of ROWS
// 128-byte rows.
template <int ROWS, int NT>
__device__ __forceinline__ void zero_chunks(uint8_t* tile, int valid) {
  for (int i = threadIdx.x; i < ROWS * 8; i += NT) {
    const int row = i >> 3, c = i & 7;
    if (c >= valid)
      *reinterpret_cast<u32x4_t*>(tile + row * kStageRow + ((c ^ swz8(row)) << 4)) = u32x4_t{0u, 0u, 0u, 0u};
  }
}

// Waits until at most X + Y * nb of this wave's copies are in flight (nb = 0 ...
// 8 weight copies per line).
template <int X, int Y>
__device__ __forceinline__ void wait_copies(int nb) {
#define SPH_WAIT(NB) asm volatile("s_waitcnt vmcnt(%0)" ::"i"(X + Y * NB < 63 ? X + Y * NB : 63) : "memory")
  if constexpr (Y == 0) {
    SPH_WAIT(0);
  } else if (nb > 4) {
    if (nb == 8) SPH_WAIT(8);
    else if (nb == 7) SPH_WAIT(7);
    else if (nb == 6) SPH_WAIT(6);
    else SPH_WAIT(5);
  } else {
    if (nb == 4) SPH_WAIT(4);
    else if (nb == 3) SPH_WAIT(3);
    else if (nb == 2) SPH_WAIT(2);
    else if (nb == 1) SPH_WAIT(1);
    else SPH_WAIT(0);
  }
#undef SPH_WAIT
}

// RA stages of h and RW of NL weight lines: step t issues h of step t + RA - 1,
// then the lines of step t + RW - 1.  LDS: [RA][h of BM rows][RW][NL][a.width
// lines rounded up to 8].
template <int BM, int BN, int WT, int RA, int RW, int NL>
__global__ __launch_bounds__(64 * stream_waves(BM)) __attribute__((amdgpu_waves_per_eu(stream_waves(BM) / 4)))
void k_mfma_stream(const MfmaArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NW = stream_waves(BM), NT = 64 * NW;
  constexpr int FR = BM / 32;  // row fragments, over as many waves as divide them
  constexpr int WN = BN == 64 ? 2 : BN == 128 ? 4 : (NW == 8 && FR % 2) ? 8 : 4;
  constexpr int WX = NW / WN;
  constexpr int WM = FR % WX == 0 ? WX : FR % 3 == 0 && WX > 3 ? 3 : FR % 2 == 0 && WX > 2 ? 2 : 1;
  constexpr int WROWS = BM / WM, WCOLS = BN / WN;        // rows and positions of a wave
  constexpr int LK = WT == 0 ? 64 : 128;                 // columns per line
  constexpr int BK = LK * NL;                            // and per stage
  constexpr int FM = WROWS / 32, FN = WCOLS / 32;
  static_assert(FM * 32 * WM == BM && FN * 32 * WN == BN && FN <= 2, "tile / waves");
  constexpr int NA = BK / 64;                            // 64-column pieces of h per stage
  constexpr int A_CP = NA * BM / 8;                      // copies of h per stage
  constexpr int A_INS = (A_CP + NW - 1) / NW, B_INS = BN / 8 / NW;  // copies per wave and stage
  static_assert(B_INS * 8 * NW == BN, "copies / waves");
  constexpr int ABYTES = NA * BM * kStageRow;
  constexpr bool kLines = RW >= 3;  // whole lines of rows that start inside one
  extern __shared__ __align__(16) uint8_t smem[];
  uint32_t* s_rmax = reinterpret_cast<uint32_t*>(smem);  // once the stages are read

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the row groups of a share of positions run next to each other on one XCD
  int nt = blockIdx.x, m0 = 0, M = a.M;
  const int K = a.K, n = a.n;
  if (a.m_tiles > 1) {
    const int c = nt / (8 * a.m_tiles), r = nt - c * 8 * a.m_tiles, shares = (n + a.width - 1) / a.width;
    const int in = min(8, shares - c * 8), per = (M + a.m_tiles - 1) / a.m_tiles;
    nt = c * 8 + r % in;
    m0 = r / in * per;
    M = min(per, M - m0);
  }
  const uint16_t* h = a.h + (int64_t)m0 * a.ldh;
  const int n0 = nt * a.width, w = min(a.width, n - n0);
  const int nsteps = (K + BK - 1) / BK, klines = (K + LK - 1) / LK;
  const int kch = K / (WT == 0 ? 8 : 16);  // 16-byte chunks of a weight row
  // rows start on a line, or stages t and t + 1 hold the columns of step t
  const bool aligned = ((reinterpret_cast<uintptr_t>(a.w) | (uint64_t)a.ldw_bytes) & 127) == 0;
  const int ahead = kLines && !aligned ? 1 : 0;
  const int nlines = nsteps > 0 ? nsteps + ahead : 0;  // stages of the weights
  const int groups = (w + 7) / 8;                 // weight copies per line
  const int nb = (groups - wave + NW - 1) / NW;   // this wave's
  const int wbytes = (a.width + 7) / 8 * 1024;    // a line of the block's rows
  const int sbytes = NL * wbytes;                 // a stage of them
  const int wn = wave % WN, wm = wave / WN;

  // copy q of a stage's NA * BM / 8 copies of h fills 8 rows; wave w issues
  // copies w, w + NW, ...; likewise the weight copies
  const int lr = lane >> 3;
  const uint8_t *pa[A_INS], *pb[B_INS];  // the lane's chunk of line 0
  int mb[B_INS];                         // chunks between the line's start and the row's
  // (a wave left without a copy of h repeats the last one: equal counts)
  auto acp = [&](int i) { return min(i * NW + wave, A_CP - 1); };
  auto chunk_of = [&](int row) { return (lane & 7) ^ swz8(row); };
#pragma unroll
  for (int i = 0; i < B_INS; ++i) {
    const int r = (i * NW + wave) * 8 + lr;
    const int id = a.ids[n0 + min(r, w - 1)];  // rows past the block's repeat its last one
    const uint8_t* row = a.w + (int64_t)id * a.ldw_bytes;
    mb[i] = ahead ? (int)((reinterpret_cast<uintptr_t>(row) & 127) >> 4) : 0;
    pb[i] = row + (chunk_of(r) - mb[i]) * 16;
  }
#pragma unroll
  for (int i = 0; i < A_INS; ++i) {
    const int g = acp(i) * 8, r = g % BM + lr, p = g / BM;
    pa[i] = reinterpret_cast<const uint8_t*>(h) + (int64_t)min(r, M - 1) * a.ldh * 2 + p * 128 + chunk_of(r) * 16;
  }
  // h of a step / line of the weights into a stage; lanes without a chunk
  // there (before the row's start, at or past its end) read the nearest one
  // the row has
  auto put = [&](const uint8_t* src, uint8_t* dst, auto ntc) {
    __builtin_amdgcn_global_load_lds(src, (lds_void_t*)dst, 16, 0, decltype(ntc)::value);
  };
  using Plain = std::integral_constant<int, 0>;
  using Nt = std::integral_constant<int, 2>;
  auto issueA = [&](int step, int stage) {
    uint8_t* as = smem + stage * ABYTES;
    const int64_t ka = (int64_t)step * BK * 2;
    if (step + 1 < nsteps) {
#pragma unroll
      for (int i = 0; i < A_INS; ++i) put(pa[i] + ka, as + acp(i) * 1024, Plain{});
    } else {
#pragma unroll
      for (int i = 0; i < A_INS; ++i) {
        const int g = acp(i) * 8, c = g / BM * 8 + chunk_of(g % BM + lr);
        put(pa[i] + (min(step * (BK / 8) + c, K / 8 - 1) - c) * 16, as + acp(i) * 1024, Plain{});
      }
    }
  };
  auto issueB = [&](int st, int stage) {
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      const int line = st * NL + l;
      uint8_t* bs = smem + RA * ABYTES + stage * sbytes + l * wbytes;
      const int64_t kb = (int64_t)line * kStageRow;
      if (line + 1 < klines && (line > 0 || !ahead)) {
#pragma unroll
        for (int i = 0; i < B_INS; ++i)
          if (i < nb) {
            if (kLines || aligned) put(pb[i] + kb, bs + (i * NW + wave) * 1024, Nt{});
            else put(pb[i] + kb, bs + (i * NW + wave) * 1024, Plain{});
          }
      } else {
#pragma unroll
        for (int i = 0; i < B_INS; ++i)
          if (i < nb) {
            const int c = chunk_of((i * NW + wave) * 8 + lr) - mb[i];
            put(pb[i] + (min(max(line * 8 + c, 0), kch - 1) - c) * 16, bs + (i * NW + wave) * 1024, Plain{});
          }
      }
    }
  };

  // fragment addresses: row (lane & 31) of a fragment; rows 32 apart share
  // the swizzle.  Sub-step p is 16 columns: chunks 2 p + lane / 32 of a bf16
  // row (64 columns per tile row), bytes 8 (lane / 32) of chunk p of an E4M3
  // row.  A weight row's chunk c lies in line (c + its offset) / 8 of stage t,
  // or past its lines in the first of stage t + 1 (bit 0 of adB; the addresses
  // are multiples of 8).
  constexpr int NP = BK / 16;                     // sub-steps of a stage
  constexpr int NK = FM + FN <= 3 ? 4 : 2;        // of which one wait covers
  uint32_t adA[NP], adB[NP][FN];
  const int hh = lane >> 5;
  {
    const int sw = swz8(lane & 31);
    const uint32_t base = (uint32_t)(uintptr_t)(lds_cptr_t)smem;
    const uint32_t ra = base + (uint32_t)(wm * WROWS + (lane & 31)) * kStageRow;
    int mis[FN];
    uint32_t rb[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      // (a row past the block's: any in LDS, its sums are not used)
      const int r = min(wn * WCOLS + j * 32 + (lane & 31), groups * 8 - 1);
      rb[j] = base + RA * ABYTES + (uint32_t)r * kStageRow;
      mis[j] = 0;
      if (ahead) {
        const uint8_t* row = a.w + (int64_t)a.ids[n0 + min(r, w - 1)] * a.ldw_bytes;
        mis[j] = (int)((reinterpret_cast<uintptr_t>(row) & 127) >> 4);
      }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      adA[p] = ra + (uint32_t)((p >> 2) * BM * kStageRow) + (uint32_t)(((2 * (p & 3) + hh) ^ sw) << 4);
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int c = (WT == 0 ? 2 * p + hh : p) + mis[j];
        adB[p][j] = (rb[j] + (c >= 8 * NL ? 0u : (uint32_t)((c >> 3) * wbytes)) + (uint32_t)(((c & 7) ^ sw) << 4) +
                     (WT == 0 ? 0u : 8u * hh)) | (c >= 8 * NL ? 1u : 0u);
      }
    }
  }

  f32x16_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // (a wave without positions computes on what the LDS holds: a branch around
  // the MFMAs made the compiler move the accumulators between register files
  // every step, 125 against 89 us for 128 rows x 60000)
  const bool busy = wm < WM && wn * WCOLS < w;
  // the first steps, in the order that the loop's counts assume: h of step
  // t + RA - 1 before line t + RW - 1, for t = -(max(RA, RW) - 1) ... -1
  constexpr int RX = RA > RW ? RA : RW;
#pragma unroll
  for (int t = 1 - RX; t < 0; ++t) {
    if (t + RA - 1 >= 0 && t + RA - 1 < nsteps) issueA(t + RA - 1, t + RA - 1);
    if (t + RW - 1 >= 0 && t + RW - 1 < nlines) issueB(t + RW - 1, t + RW - 1);
  }
  int sa = 0, fa = RA - 1, sb = 0, fb = RW - 1;  // stages read and filled
  for (int t = 0; t < nsteps; ++t) {
    // this wave's copies of h(t) and lines t (and t + 1) have landed, younger
    // ones may be in flight: those after h(t) are RA - 2 whole steps and one
    // line, those after line t + ahead are RW - 2 - ahead whole steps.  Past
    // the barrier every wave's have landed, and every wave has read step t - 1.
    constexpr int D0 = RW - 2 < RA - 1 ? RW - 2 : RA - 1, D1 = RW - 3 < RA - 1 ? RW - 3 : RA - 1;
    // (D = RA - 1 whole steps less the first one's h)
    constexpr int X0 = (D0 == RA - 1 ? D0 - 1 : D0) * A_INS, X1 = D1 < 0 ? 0 : (D1 == RA - 1 ? D1 - 1 : D1) * A_INS;
    if (t + RX - 1 >= nsteps) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (kLines && ahead) wait_copies<X1, D1 < 0 ? 0 : D1 * NL>(nb);
    else wait_copies<X0, D0 * NL>(nb);
    __builtin_amdgcn_s_barrier();
    if (t + RA - 1 < nsteps) issueA(t + RA - 1, fa);
    if (t + RW - 1 < nlines) issueB(t + RW - 1, fb);
    const int left = K - t * BK;  // columns from step t on
    const int nextb = sb + 1 == RW ? 0 : sb + 1;
    const uint32_t oa = (uint32_t)(sa * ABYTES), so = (uint32_t)(sb * sbytes), sn = (uint32_t)(nextb * sbytes);
    const bool tail = left < BK;
    if (tail) {
      // columns past K: zeros in h
      uint8_t* as = smem + sa * ABYTES;
#pragma unroll
      for (int p = 0; p < NA; ++p) zero_chunks<BM, NT>(as + p * BM * kStageRow, max(0, left / 8 - 8 * p));
      __syncthreads();
    }
    {
      typedef ReadFrags<FM, FN, NK, WT> Read;
#pragma unroll
      for (int p0 = 0; p0 < NP; p0 += NK) {
        uint32_t pa_[NK], pb_[NK][FN];
        u32x4_t af[NK][FM];
        typename Read::B bf[NK][FN];
#pragma unroll
        for (int s = 0; s < NK; ++s) {
          const int p = p0 + s;
          pa_[s] = adA[p] + oa;
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            pb_[s][j] = (adB[p][j] & ~1u) + ((adB[p][j] & 1u) ? sn : so);
            // columns past K: the weights' lanes read the zeros of h
            if (tail && 16 * p + 8 * hh >= left) pb_[s][j] = pa_[s];
          }
        }
        Read::run(af, bf, pa_, pb_);
#pragma unroll
        for (int s = 0; s < NK; ++s) {
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            u32x4_t wv;
            if constexpr (WT == 0) {
              wv = bf[s][j];
            } else {
              wv.x = e4m3x2_to_bf16x2_m<false>(bf[s][j].x);
              wv.y = e4m3x2_to_bf16x2_m<true>(bf[s][j].x);
              wv.z = e4m3x2_to_bf16x2_m<false>(bf[s][j].y);
              wv.w = e4m3x2_to_bf16x2_m<true>(bf[s][j].y);
            }
#pragma unroll
            for (int i = 0; i < FM; ++i)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, af[s][i]),
                                                                  __builtin_bit_cast(bf16x8_t, wv),
                                                                  acc[i][j], 0, 0, 0);
          }
        }
      }
    }
    sa = sa + 1 == RA ? 0 : sa + 1;
    fa = fa + 1 == RA ? 0 : fa + 1;
    sb = nextb;
    fb = fb + 1 == RW ? 0 : fb + 1;
  }
  __syncthreads();  // the stages are read
  for (int i = tid; i < BM; i += NT) s_rmax[i] = 0u;
  __syncthreads();

  // Epilogue: z through a buffer descriptor of its rows, so that rows past M,
  // and positions past the block's at an offset beyond it, are dropped by the
  // store itself; max |clamp(z)| = min(|z|, c).
  constexpr int P = (FM * 16 + 31) / 32 * 32;
  if (busy) {
    float red[P];
#pragma unroll
    for (int t = 0; t < P; ++t) red[t] = 0.0f;
    const float clip = a.clip;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(scalar_ptr(a.z + (int64_t)m0 * a.ldz)), 0,
                                                        (int)((uint32_t)M * (uint32_t)a.ldz * 4u), 0x00020000);
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int rel = wn * WCOLS + j * 32 + (lane & 31);
      const int col = n0 + rel;
      const int id = a.ids[n0 + min(rel, w - 1)];
      float cs = 1.0f;
      if constexpr (WT == 1) cs = a.wscale[id];
      const bool hb = a.bias != nullptr;
      const float cb = hb ? a.bias[id] : 0.0f;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float zv = cloud_value<WT>(acc[i][j][r], cs, hb, cb);
          const uint32_t row = (uint32_t)(wm * WROWS + i * 32 + 8 * (r >> 2) + 4 * hh + (r & 3));
          const uint32_t off = rel < w ? (row * (uint32_t)a.ldz + (uint32_t)col) * 4u : 0xF0000000u;
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(zv), rsrc, (int)off, 0, 0);
          red[i * 16 + r] = fmaxf(red[i * 16 + r], rel < w ? fminf(fabsf(zv), clip) : 0.0f);
        }
      }
    }
    half_wave_max_transpose<P>(red, lane);
    constexpr int PER = P / 32;
#pragma unroll
    for (int t = 0; t < PER; ++t) {
      const int idx = (lane & 31) * PER + t;
      if (idx >= FM * 16) continue;
      const int i = idx / 16, r = idx % 16;
      atomicMax(&s_rmax[wm * WROWS + i * 32 + 8 * (r >> 2) + 4 * hh + (r & 3)], __float_as_uint(red[t]));
    }
  }
  __syncthreads();
  for (int i = tid; i < BM; i += NT)
    if (i < M) a.amax_part[(int64_t)(m0 + i) * kMaxBlocks + nt] = __uint_as_float(s_rmax[i]);
#endif
}

template <int BM, int BN, int WT, int RA, int RW, int NL>
static hipError_t launch_stream_tile(const MfmaArgs& a, hipStream_t s) {
  static std::atomic<uint64_t> lds_set{0};
  constexpr int abytes = BM * (WT == 0 ? 1 : 2) * NL * kStageRow;
  constexpr size_t most = std::min((size_t)kLdsBytes, (size_t)RA * abytes + (size_t)RW * NL * BN * kStageRow);
  const size_t lds = (size_t)RA * abytes + (size_t)RW * NL * ((a.width + 7) / 8 * 1024);
  if (lds > most || a.width > BN) return hipErrorInvalidValue;
  auto k = k_mfma_stream<BM, BN, WT, RA, RW, NL>;
  hipError_t e = set_lds_limit_once(lds_set, reinterpret_cast<const void*>(k), most);
  if (e != hipSuccess) return e;
  launch_kernel(k, dim3((a.n + a.width - 1) / a.width * a.m_tiles), dim3(64 * stream_waves(BM)), lds, s, a);
  return hipGetLastError();
}

// Row groups of the streaming kernel, 0 where the tiles of launch_mfma are the
// faster way.  More than kStreamMaxRows rows are split into 2, 4 or 8 groups
// (the CUs divide evenly) where 256-position tiles would leave half of the CUs
// or more without work and the groups' shares fit one round.  (us, tiles /
// groups, K 3584 ... 4032: 256 rows x 8000 69 / 36, 320 x 15000 99 / 65, 320 x
// 30000 103 / 93, 400 x 16000 85 / 75, 640 x 8000 88 / 64, 640 x 16000 107 /
// 100, 1024 x 8000 83 / 76, E4M3 268 x 30000 116 / 93, 512 x 8000 83 / 47; past
// the rule 384 x 32000 105 / 111, 768 x 16000 95 / 103, 1280 x 6000 78 / 85.)
int stream_groups(int M, int n) {
  if (M <= kStreamMaxRows) return 1;
  int g = 2;
  while (g * kStreamMaxRows < M) g *= 2;
  return M <= 1024 && mfma_tiles(M, n) <= kCUs / 2 && (int64_t)n * g <= kCUs * 256 ? g : 0;
}

// Positions per block: an equal share for every CU of a row group, in as many
// rounds as 256 positions per block need, at least 32 (a fragment).
int stream_width(int M, int n) {
  const int cus = kCUs / std::max(1, stream_groups(M, n));
  const int rounds = (n + cus * 256 - 1) / (cus * 256);
  const int w = (n + cus * rounds - 1) / (cus * rounds);
  return w < 32 ? 32 : w;
}

// Stages by what fits: as many lines as possible, at least two of h.  Narrow
// blocks take two lines a stage where three such stages fit: with little to copy
// and multiply a step is the barrier's and the fragment reads' latency (0.5 us
// for 18 rows), so half as many are faster.  (us, one line / two: 18 rows x
// 14464 x 7680 columns 66 / 51, 60 x 30000 x 3584 45 / 40, 90 x 8000 x 3584 40 /
// 30, 256 x 8000 x 3584 in two groups 42 / 36, E4M3 30 x 5000 x 8128 52 / 41.)
template <int BM_, int BN_, int RA_, int RW_, int NL_ = 1>
struct StreamTile {
  static constexpr int BM = BM_, BN = BN_, RA = RA_, RW = RW_, NL = NL_;
};

// f(StreamTile<...>{}) of the instance for row tile BM and this width
template <int BM, int WT, class F>
static hipError_t with_stream_tile(int width, F f) {
  constexpr int ak = BM * (WT == 0 ? 1 : 2) / 8;  // KB of a stage of h
  if constexpr (BM != 160) {  // (with_stream_rows: other row counts)
    if (width <= 64) {
      constexpr int r = std::min(8, 160 / (ak + 8)), r2 = std::min(8, 160 / (2 * (ak + 8)));
      if constexpr (r2 >= 3) return f(StreamTile<BM, 64, r2, r2, 2>{});
      else return f(StreamTile<BM, 64, r, r>{});
    }
  }
  if constexpr (BM != 160 && BM != 96) {
    if (width <= 128) {
      constexpr int r = std::min(6, 160 / (ak + 16)), r2 = std::min(6, 160 / (2 * (ak + 16)));
      if constexpr (r2 >= 3) return f(StreamTile<BM, 128, r2, r2, 2>{});
      else return f(StreamTile<BM, 128, r, r>{});
    }
  }
  if constexpr (4 * (ak + 32) <= 160) {
    return f(StreamTile<BM, 256, 4, 4>{});
  } else {
    if (2 * ak + 4 * ((width + 7) / 8) <= 160) return f(StreamTile<BM, 256, 2, 4>{});
    if constexpr (3 * (ak + 32) <= 160) return f(StreamTile<BM, 256, 3, 3>{});
    if (2 * ak + 3 * ((width + 7) / 8) <= 160) return f(StreamTile<BM, 256, 2, 3>{});
    return f(StreamTile<BM, 256, 2, 2>{});
  }
}

// Blocks of at most 128 positions have more than one row of waves: 3 and 5
// row fragments, which it does not divide, run as 4 and 6 (but 3 over four
// rows of waves, at most 64 positions).  155 rows x 16000 x 3584 columns 85 ->
// 54 us, x 30000 x 4000 102 -> 78; 90 x 30000 x 3584 64 -> 56.
template <int WT, class F>
static hipError_t with_stream_rows(int M, int groups, int width, F f) {
  int fr = ((M + groups - 1) / groups + 31) / 32;
  if (width <= 128 && (fr == 5 || (fr == 3 && width > 64))) ++fr;
  switch (fr) {
    case 1: return with_stream_tile<32, WT>(width, f);
    case 2: return with_stream_tile<64, WT>(width, f);
    case 3: return with_stream_tile<96, WT>(width, f);
    case 4: return with_stream_tile<128, WT>(width, f);
    case 5: return with_stream_tile<160, WT>(width, f);
    default: return with_stream_tile<192, WT>(width, f);
  }
}

template <int WT>
static hipError_t launch_stream_rows(const MfmaArgs& a, hipStream_t s) {
  return with_stream_rows<WT>(a.M, a.m_tiles, a.width, [&](auto t) {
    using T = decltype(t);
    return launch_stream_tile<T::BM, T::BN, WT, T::RA, T::RW, T::NL>(a, s);
  });
}

void stream_tile(int M, int n, int wtype, int tile[5]) {
  auto put = [&](auto t) {
    using T = decltype(t);
    const int v[5] = {T::BM, T::BN, T::RA, T::RW, T::NL};
    std::copy(v, v + 5, tile);
    return hipSuccess;
  };
  const int g = std::max(1, stream_groups(M, n)), w = stream_width(M, n);
  (void)(wtype == 0 ? with_stream_rows<0>(M, g, w, put) : with_stream_rows<1>(M, g, w, put));
}

hipError_t launch_stream(int wtype, MfmaArgs a, hipStream_t s) {
  a.width = stream_width(a.M, a.n);
  a.m_tiles = stream_groups(a.M, a.n);
  const int blocks = (a.n + a.width - 1) / a.width;
  if (a.M < 1 || a.m_tiles < 1 || blocks > kMaxBlocks || a.K % (wtype == 0 ? 8 : 16) != 0)
    return hipErrorInvalidValue;
  return wtype == 0 ? launch_stream_rows<0>(a, s) : launch_stream_rows<1>(a, s);
}

}  // namespace sph
