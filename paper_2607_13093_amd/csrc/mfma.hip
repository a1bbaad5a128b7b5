// Dense gathered projection for many rows of h (MFMA path).
//
//   C[m, j] = sum_k h[m, k] * W[S_j, k]      (eq. 12 on the subset S)
//
// With hundreds of rows the contraction is dense enough for the matrix
// cores: a block computes a BM x BN tile of C with v_mfma_f32_32x32x16_bf16
// (bf16 inputs, fp32 accumulation).  Both operands are K-contiguous in
// memory (h is [M, K] row-major, the weight rows are vocab-major), and both
// tiles are copied global-to-LDS as [rows][BK].  The B tile is gathered: tile
// column j is weight row S[n0 + j]; fp8 E4M3 rows are widened to bf16
// (exactly) in registers and their per-row scale is applied in the epilogue.
// Any K that is whole 16-byte chunks takes these kernels: staging partial
// steps through registers instead ran 3 to 5 times slower (268 rows x 15360 x
// 4048 columns 172 us, see TAIL).
//
// Operand layouts of the 32x32x16 instruction (checked on the hardware):
//   A: lane l supplies A[l % 32][8 * (l / 32) + e], e = 0..7
//   B: lane l supplies B[8 * (l / 32) + e][l % 32]
//   C: accumulator r of lane l is C[8 * (r / 4) + 4 * (l / 32) + r % 4][l % 32]
//
// Tile order: blocks are dealt round-robin to the 8 XCDs, so block b is
// remapped to give each XCD a contiguous range of tiles, and tiles are
// numbered with the m-tiles of one n-tile adjacent (groups of up to GM):
// blocks sharing a gathered B tile (or an A panel) run on the same XCD at the
// same time and meet in its L2.
//
// Epilogue: scales fp8 columns, adds the bias, writes fp32 partial logits and
// the tile's row maxima of |clamp(z)|.  (The endpoint projection has its own
// kernel.)
#include "mfma_tile.h"

namespace sph {

// Descriptor of `rows` rows of z from the tile's first one (at most 320 rows of
// 2^19 positions, below 2^30 bytes), an offset past any tile's, and the
// non-temporal store of one value.
__device__ __forceinline__ auto tile_rsrc(float* z, int rows, int ldz) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(scalar_ptr(z)), 0,
                                           (int)((uint32_t)rows * (uint32_t)ldz * 4u), 0x00020000);
}
constexpr uint32_t kPastTile = 0xC0000000u;  // (plus an offset inside the tile: no wrap)
__device__ __forceinline__ void store_z(float v, __amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rsrc, (int)off, 0, 2);
}

// From the row of accumulator r - 1 (of the previous fragment for r = 0) to that
// of r: the next row, or the fifth next.  The empty asm keeps one running
// offset: all of them at once spilled 100 registers.
__device__ __forceinline__ void next_row(uint32_t& off, int r, int ldz) {
  off += (uint32_t)ldz * (r % 4 == 0 ? 20u : 4u);
  asm volatile("" : "+v"(off));
}

// Epilogue of a BM x BN tile held as acc[FM][FN] 32x32 fragments by the
// WM x WN waves.  Row of accumulator r in fragment (i, j):
// 8*(r/4) + 4*(lane/32) + r%4; column: lane % 32.
// s_q: LDS the main loop no longer needs (BM*BN bytes; kEpiCloudQ only).  The
// caller has passed a barrier after its last LDS read.
template <int BM, int BN, int WM, int WN, int WT, int EPI, int FM, int FN>
__device__ __forceinline__ void tile_epilogue(f32x16_t (&acc)[FM][FN], const MfmaArgs& a,
                                              const int32_t* s_ids, uint32_t* s_rmax, int m0,
                                              int n0, int nt, int8_t* s_q) {
  constexpr int NT = 64 * WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int P = (FM * 16 + 31) / 32 * 32;  // row values per lane, padded for the butterfly
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int M = a.M, n = a.n, ldz = a.ldz;
  float red[P];
#pragma unroll
  for (int t = FM * 16; t < P; ++t) red[t] = 0.0f;
  // z goes out through a buffer descriptor of the tile's rows: a store past
  // row M - 1 is dropped, so every tile inside the positions runs the same
  // straight-line code, and in the last one the lanes past n store beyond the
  // descriptor.  Rows past M and positions past n repeat a valid one, so they
  // leave the maxima as they are; max |clamp(z)| is taken as min(|z|, c), which
  // is the same value for every z, NaN included.  (A bounds test per element
  // compiled to two branches, a 64-bit address and a reload of the bias
  // pointer: 13.6 us of a 210 us block on the dense 2048-row shape, now 7, and
  // every tile of a batch whose rows do not fill its row tiles.)
  const auto rsrc = tile_rsrc(a.z ? a.z + (int64_t)m0 * ldz : nullptr, min(BM, M - m0), ldz);
  const uint32_t lrow0 = (uint32_t)(wm * TM + 4 * (lane >> 5));
  const uint32_t lcol0 = (uint32_t)(n0 + wn * TN + (lane & 31));
  auto fill = [&](auto edge, auto has_bias, auto store) {
    constexpr bool ED = decltype(edge)::value, HB = decltype(has_bias)::value, ST = decltype(store)::value;
    float cs[FN], cb[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int id = s_ids[wn * TN + j * 32 + (lane & 31)];
      cs[j] = WT == 1 ? a.wscale[id] : 1.0f;
      cb[j] = HB && a.bias ? a.bias[id] : 0.0f;
    }
    const bool hb = a.bias != nullptr;
    uint32_t oj[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) oj[j] = ED && lcol0 + 32u * j >= (uint32_t)n ? kPastTile : 128u * j;
    const float clip = a.clip;
    uint32_t off = (lrow0 * (uint32_t)ldz + lcol0) * 4u;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (i + r > 0) next_row(off, r, ldz);
        float best = 0.0f;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const float zv = cloud_value<WT>(acc[i][j][r], cs[j], HB && hb, cb[j]);
          if constexpr (ST) store_z(zv, rsrc, off + oj[j]);
          best = fmaxf(best, fminf(fabsf(zv), clip));
        }
        red[i * 16 + r] = best;
      }
    }
  };
  {
    using T = std::true_type;
    using F = std::false_type;
    const bool st = EPI == kEpiCloud || a.z != nullptr, edge = n0 + BN > n;
    if (!st) {
      if (a.bias) fill(F{}, T{}, F{});
      else fill(F{}, F{}, F{});
    } else if (edge) {
      fill(T{}, T{}, T{});
    } else if (a.bias) {
      fill(F{}, T{}, T{});
    } else {
      fill(F{}, F{}, T{});
    }
  }
  half_wave_max_transpose<P>(red, lane);
  constexpr int PER = P / 32;
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int idx = (lane & 31) * PER + t;
    if (idx >= FM * 16) continue;
    const int i = idx / 16, r = idx % 16;
    const int lrow = wm * TM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    atomicMax(&s_rmax[lrow], __float_as_uint(red[t]));
  }
  __syncthreads();
  if constexpr (EPI == kEpiCloudQ) {
    // The tile is one scale block of every row: s = a / qmax from the tile's
    // row maximum of |clamp(z)|, codes rint(clamp(z) / s) from the
    // accumulators still in registers (the same fp32 operations as the
    // quantiser kernel), one byte per code in LDS (the A staging area), then
    // stored row by row, two codes per byte for b = 4; codes of positions
    // past n are 0 (the pad nibble).
    const float qmax = a.qout_bits == 8 ? 127.0f : 7.0f;
    float cs[FN], cb[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int id = s_ids[wn * TN + j * 32 + (lane & 31)];
      cs[j] = WT == 1 ? a.wscale[id] : 1.0f;
      cb[j] = a.bias ? a.bias[id] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int lrow = wm * TM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const float sc = __uint_as_float(s_rmax[lrow]) / qmax;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int lcol = wn * TN + j * 32 + (lane & 31);
          int code = 0;
          if (n0 + lcol < n) {
            // (without a bias 0 is added, which changes no code)
            const float zq = cloud_value<WT>(acc[i][j][r], cs[j], true, cb[j]);
            const float y = fminf(fmaxf(zq, -a.clip), a.clip);
            const float t = sc > 0.0f ? y / sc : 0.0f;
            code = (int)fminf(fmaxf(rintf(t), -qmax), qmax);
          }
          s_q[lrow * BN + lcol] = (int8_t)code;
        }
      }
    }
    __syncthreads();
    const int bits = a.qout_bits;
    const int TB = BN * bits / 8;                      // code bytes of a tile row
    const int64_t c0 = (int64_t)n0 * bits / 8;
    const int64_t rowbytes = ((int64_t)n * bits + 7) / 8;
    const bool vec = (a.qout_stride & 15) == 0 && (reinterpret_cast<uintptr_t>(a.qout) & 15) == 0;
    for (int c = tid; c < BM * (TB / 16); c += NT) {
      const int r = c / (TB / 16), k = c % (TB / 16);
      const int row = m0 + r;
      const int64_t col = c0 + (int64_t)k * 16;
      if (row >= M || col >= rowbytes) continue;
      uint32_t wv[4];
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        uint32_t w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int byte = 4 * e4 + e;
          uint32_t v;
          if (bits == 8) {
            v = (uint8_t)s_q[r * BN + k * 16 + byte];
          } else {
            const int p0 = k * 32 + 2 * byte;
            v = ((uint32_t)s_q[r * BN + p0] & 15u) | (((uint32_t)s_q[r * BN + p0 + 1] & 15u) << 4);
          }
          w |= v << (8 * e);
        }
        wv[e4] = w;
      }
      uint8_t* dst = a.qout + (int64_t)row * a.qout_stride + col;
      if (vec && col + 16 <= rowbytes) {
        *reinterpret_cast<u32x4_t*>(dst) = u32x4_t{wv[0], wv[1], wv[2], wv[3]};
      } else {
        for (int b = 0; b < 16 && col + b < rowbytes; ++b) dst[b] = (uint8_t)(wv[b >> 2] >> (8 * (b & 3)));
      }
    }
    for (int i = tid; i < BM; i += NT) {
      const int row = m0 + i;
      if (row < M) a.qout_scale[(int64_t)row * a.qout_nb + nt] = __uint_as_float(s_rmax[i]) / qmax;
    }
    return;
  }
  for (int i = tid; i < BM; i += NT) {
    const int row = m0 + i;
    if (row < M) a.amax_part[(int64_t)row * kMaxBlocks + nt] = __uint_as_float(s_rmax[i]);
  }
}

// Tiles of bf16 weights, K a multiple of 8 (TAIL: no multiple of the K step;
// the missing chunks of the last step read its first chunk and are cleared in
// LDS).  gfx950's global_load_lds_dwordx4 writes a wave's 64 x 16 bytes straight into LDS
// (lane l at base + 16*l), so tiles never pass through registers and no
// ds_write is issued.  A wave instruction fills 8 rows x 128 bytes; rows are
// unpadded and their 16-byte chunks are XOR-swizzled with
// f(row) = (row & 7) ^ ((row >> 3) & 1), which keeps every fragment read
// conflict-free whether the LDS serves 8 or 16 lanes per cycle.  Rows past
// M and subset positions past n read a valid row (row M-1 / the last id):
// they only feed outputs that are never written.  On the decode-sized dense
// shape this loop ran 1.2x faster than register staging.
// Waves: WM x WN (wave tile (BM/WM) x (BN/WN)), two per SIMD, whose
// accumulators live in the 256 registers each wave has.
template <int BM, int BN, int WM, int WN, int EPI, bool O32, bool TAIL>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(WM * WN / 4, WM * WN / 4)))
void k_mfma_dma(const MfmaArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NT = 64 * WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / 32, FN = TN / 32;
  // Only the first wave of each SIMD issues the
  // copies (all of them): a copy instruction can hold its wave at issue
  // until the load path accepts it, and the SIMD's other wave keeps the
  // matrix pipe busy meanwhile.  Measured on the dense 2048-row shape: 3-5%
  // faster than all 8 waves issuing an eighth of the copies each.
  constexpr int IW = WM * WN / 2;
  constexpr int A_INS = BM / 8 / IW, B_INS = BN / 8 / IW;  // copy instructions per issuing wave per step
  static_assert(A_INS * 8 * IW == BM && B_INS * 8 * IW == BN, "tile rows / issuing waves");
  extern __shared__ __align__(16) uint8_t smem[];
  uint16_t* As = reinterpret_cast<uint16_t*>(smem);      // [2][BM][64]
  uint16_t* Bs = As + 2 * BM * kBK;                       // [2][BN][64]
  int32_t* s_ids = reinterpret_cast<int32_t*>(Bs + 2 * BN * kBK);
  uint32_t* s_rmax = reinterpret_cast<uint32_t*>(s_ids + BN);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int iw = wave < IW ? wave : 0;  // issuing slot (waves >= IW issue nothing)
  const int wm = wave / WN, wn = wave % WN;
  int mt, nt;
  tile_of_block(blockIdx.x, a.m_tiles, a.n_tiles, mt, nt);
  const int m0 = mt * BM, n0 = nt * BN;
  const int M = a.M, K = a.K, n = a.n;
  const int last_id = a.ids[min(n, n0 + BN) - 1];
  for (int i = tid; i < BN; i += NT) s_ids[i] = n0 + i < n ? a.ids[n0 + i] : last_id;
  for (int i = tid; i < BM; i += NT) s_rmax[i] = 0u;
  __syncthreads();

  // lane -> row (lane / 8) of its 8-row group and the logical chunk it fetches
  const int lr = lane >> 3;
  const uint8_t* hbase = reinterpret_cast<const uint8_t*>(a.h);
  LaneAddr<O32> pa[A_INS], pb[B_INS];
#pragma unroll
  for (int i = 0; i < A_INS; ++i) {
    const int r = (iw * A_INS + i) * 8 + lr;
    const int lc = (lane & 7) ^ swz8(r);
    pa[i].set(hbase, (int64_t)min(m0 + r, M - 1) * a.ldh * 2 + lc * 16);
  }
#pragma unroll
  for (int i = 0; i < B_INS; ++i) {
    const int r = (iw * B_INS + i) * 8 + lr;
    const int lc = (lane & 7) ^ swz8(r);
    pb[i].set(a.w, (int64_t)s_ids[r] * a.ldw_bytes + lc * 16);
  }
  auto issue = [&](int k0, int stage) {
    if (wave >= IW) return;
    uint8_t* as = reinterpret_cast<uint8_t*>(As + stage * BM * kBK);
    uint8_t* bs = reinterpret_cast<uint8_t*>(Bs + stage * BN * kBK);
    const int64_t step = (int64_t)k0 * 2;
    const uint8_t* ha = O32 ? scalar_ptr(hbase + step) : nullptr;
    const uint8_t* wb = O32 ? scalar_ptr(a.w + step) : nullptr;
    if (!TAIL || K - k0 >= kBK) {
#pragma unroll
      for (int i = 0; i < A_INS; ++i) pa[i].copy(ha, step, (lds_void_t*)(as + (iw * A_INS + i) * 1024));
#pragma unroll
      for (int i = 0; i < B_INS; ++i) pb[i].copy(wb, step, (lds_void_t*)(bs + (iw * B_INS + i) * 1024));
    } else {
      const int valid = K - k0;
      auto back = [&](int r) {
        const int c = (lane & 7) ^ swz8(r);
        return c * 8 < valid ? 0u : (uint32_t)(c * 16);
      };
#pragma unroll
      for (int i = 0; i < A_INS; ++i)
        pa[i].copy_back(ha, step, (lds_void_t*)(as + (iw * A_INS + i) * 1024), back((iw * A_INS + i) * 8 + lr));
#pragma unroll
      for (int i = 0; i < B_INS; ++i)
        pb[i].copy_back(wb, step, (lds_void_t*)(bs + (iw * B_INS + i) * 1024), back((iw * B_INS + i) * 8 + lr));
    }
  };

  f32x16_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  if (K > 0) {
    issue(0, 0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }
  int stage = 0;
  for (int k0 = 0; k0 < K; k0 += kBK) {
    // the other stage was last read in the previous step, finished by all
    // waves before that step's closing barrier
    if (k0 + kBK < K) issue(k0 + kBK, stage ^ 1);
    if (TAIL && K - k0 < kBK) {
      zero_tail<BM, NT>(As + stage * BM * kBK, K - k0);
      zero_tail<BN, NT>(Bs + stage * BN * kBK, K - k0);
      __syncthreads();
    }
    const uint16_t* as = As + stage * BM * kBK;
    const uint16_t* bs = Bs + stage * BN * kBK;
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      bf16x8_t af[FM], bfr[FN];
      const int c = kk * 2 + (lane >> 5);
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int row = wm * TM + i * 32 + (lane & 31);
        af[i] = *reinterpret_cast<const bf16x8_t*>(as + row * kBK + ((c ^ swz8(row)) << 3));
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int row = wn * TN + j * 32 + (lane & 31);
        bfr[j] = *reinterpret_cast<const bf16x8_t*>(bs + row * kBK + ((c ^ swz8(row)) << 3));
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0);  // this wave's loads for the next stage have landed
    __syncthreads();
    stage ^= 1;
  }
  tile_epilogue<BM, BN, WM, WN, 0, EPI>(acc, a, s_ids, s_rmax, m0, n0, nt, reinterpret_cast<int8_t*>(As));
#endif
}

// One wave per SIMD for the dense bf16 cloud projection (256 x 256 tiles, an
// even number, at least 2, of 64-wide K steps).  Four waves, each a 128 x 128 wave tile of
// 4 x 4 fragments whose 256 accumulators stay in the AGPRs: per 16-wide
// sub-step a wave reads 8 fragments for 16 MFMAs, where the two-wave kernel
// reads 6 for 8, so the LDS traffic per flop drops by a third.  With no second
// wave on the SIMD the schedule is explicit: the MFMAs and the LDS fragment
// reads are inline asm (their order is kept as written).  Four fragment
// register sets, one per sub-step: while a sub-step's 16 MFMAs issue, the
// reads for the sub-step two ahead go out after its first 8 MFMAs, into the
// set the MFMAs of two sub-steps ago used.  One barrier per step, between the
// second and third sub-steps: the third and fourth then read the next stage
// and (two weight stages) copy the step after next into this one, 8 copies
// each; three weight stages spread the copies differently (below).  Past the end
// the copies repeat the last step (in-bounds reads into a stage nobody reads),
// so the K loop is straight-line code: with a branch in it the compiler
// spilled registers that reads still in flight were to fill.  The compiler
// sees neither the asm reads nor the MFMAs, so every wait is explicit
// (lgkmcnt before each sub-step's MFMAs, vmcnt and lgkmcnt before the
// barrier), and each sub-step's fragments stay allocated to its end.
// Measured (harness, dense_full / dense_sub): reads one sub-step ahead with
// two sets 3397 / 1022 us, two ahead with four sets 3300 / 970 us.
__device__ __forceinline__ void w1_mfma(f32x16_t& c, const bf16x8_t& a, const bf16x8_t& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
template <int OFF>
__device__ __forceinline__ void w1_read(bf16x8_t& d, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "i"(OFF));
}
__device__ __forceinline__ void w1_wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// the older of two groups of 8 reads (LDS reads complete in order)
__device__ __forceinline__ void w1_wait_lds8() { asm volatile("s_waitcnt lgkmcnt(8)" ::: "memory"); }
__device__ __forceinline__ void w1_wait_mem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
typedef __attribute__((address_space(3))) const char* lds_cptr_t;

// NB weight stages: 2 (an even number of K steps; 128 KB of LDS), or 3 (a
// multiple of 6 steps; all 160 KB of LDS, and the ids and row maxima live
// outside the stages: ids are read from global memory, the row maxima take
// the first stage after the K loop).  With three, a step's first two
// sub-steps copy the weights of two steps ahead into the stage the previous
// step read and its last two copy h, one copy per 4 MFMAs in every sub-step,
// so the barrier waits for all but the newest 8 copies (those weights).
// Harness, dense_full / dense_sub: two stages 3300 / 996 us; three, weights
// copied in the last sub-step three steps ahead, 3250 / 970 us; three with
// the copies spread over the step 3290 -> 3257 / 1004 -> 961 us (A/B runs).
// Odd or partial last steps run on k_mfma_dma (an epilogue for them here was no
// faster: 1184 rows x 31038 x 4000 columns 400 against 390 us, 1999 x 32767 x
// 4032 567 against 526).
template <int EPI, int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void k_mfma_w1(const MfmaArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  static_assert(EPI == kEpiCloud, "cloud epilogue only");
  static_assert(NB == 2 || NB == 3, "two or three weight stages");
  constexpr int BM = 256, BN = 256, NT = 256, WN = 2, TM = 128, TN = 128, FM = 4, FN = 4;
  constexpr int A_INS = BM / 8 / 4, B_INS = BN / 8 / 4;  // 8 + 8 copies per wave per step
  constexpr int SB = BN * kBK * 2;                        // bytes of a stage (32 KB)
  extern __shared__ __align__(16) uint8_t smem[];
  uint8_t* As = smem;                                     // [2][256][128 B]
  uint8_t* Bs = smem + 2 * SB;                            // [NB][256][128 B]
  // ids and row maxima: after the stages (NB = 2), or none / the first stage
  // once the K loop is done (NB = 3)
  int32_t* s_ids = reinterpret_cast<int32_t*>(Bs + NB * SB);
  uint32_t* s_rmax = NB == 2 ? reinterpret_cast<uint32_t*>(s_ids + BN) : reinterpret_cast<uint32_t*>(smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  int mt, nt;
  tile_of_block(blockIdx.x, a.m_tiles, a.n_tiles, mt, nt);
  const int m0 = mt * BM, n0 = nt * BN;
  const int M = a.M, K = a.K, n = a.n;
  const int S = K / kBK;  // a multiple of 2 (NB = 2) or 6 (NB = 3): the launcher's condition
  const int last_id = a.ids[min(n, n0 + BN) - 1];
  if constexpr (NB == 2) {
    for (int i = tid; i < BN; i += NT) s_ids[i] = n0 + i < n ? a.ids[n0 + i] : last_id;
    for (int i = tid; i < BM; i += NT) s_rmax[i] = 0u;
    __syncthreads();
  }

  const int lr = lane >> 3;
  const uint8_t* hbase = reinterpret_cast<const uint8_t*>(a.h);
  LaneAddr<true> pa[A_INS], pb[B_INS];
#pragma unroll
  for (int i = 0; i < A_INS; ++i) {
    const int r = (wave * A_INS + i) * 8 + lr;
    const int lc = (lane & 7) ^ swz8(r);
    pa[i].set(hbase, (int64_t)min(m0 + r, M - 1) * a.ldh * 2 + lc * 16);
  }
#pragma unroll
  for (int i = 0; i < B_INS; ++i) {
    const int r = (wave * B_INS + i) * 8 + lr;
    const int lc = (lane & 7) ^ swz8(r);
    const int id = NB == 2 ? s_ids[r] : (n0 + r < n ? a.ids[n0 + r] : last_id);
    pb[i].set(a.w, (int64_t)id * a.ldw_bytes + lc * 16);
  }
  // copy i (0..7) of this wave's share of step s into stage st
  auto copyA = [&](int i, int s, int st) {
    const int64_t step = (int64_t)s * kBK * 2;
    pa[i].copy(scalar_ptr(hbase + step), step, (lds_void_t*)(As + st * SB + (wave * A_INS + i) * 1024));
  };
  auto copyB = [&](int i, int s, int st) {
    const int64_t step = (int64_t)s * kBK * 2;
    pb[i].copy(scalar_ptr(a.w + step), step, (lds_void_t*)(Bs + st * SB + (wave * B_INS + i) * 1024));
  };
  // fragment reads: row (lane & 31) of a fragment, 16-byte chunk 2 kk + lane / 32
  // (swizzled); the fragments of a wave are 32 rows (4 KB) apart and the
  // stages 32 KB apart, both immediate offsets of the read (the third weight
  // stage, past the 16-bit offset field, has base addresses of its own)
  uint32_t adA[4], adB[4], adB2[4];
  {
    const int sw = swz8(lane & 31);  // rows 32 apart share the swizzle
    const uint32_t baseA = (uint32_t)(uintptr_t)(lds_cptr_t)As + (uint32_t)((wm * TM + (lane & 31)) * 128);
    const uint32_t baseB = (uint32_t)(uintptr_t)(lds_cptr_t)Bs + (uint32_t)((wn * TN + (lane & 31)) * 128);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const uint32_t c = (uint32_t)(((kk * 2 + (lane >> 5)) ^ sw) << 4);
      adA[kk] = baseA + c;
      adB[kk] = baseB + c;
      adB2[kk] = baseB + 2u * SB + c;
    }
  }
  f32x16_t acc[FM][FN];
  {
    f32x16_t z0;
#pragma unroll
    for (int r = 0; r < 16; ++r) z0[r] = 0.0f;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) asm volatile("; zero accumulators" : "=a"(acc[i][j]) : "0"(z0));
  }
  bf16x8_t f0a[FM], f0b[FN], f1a[FM], f1b[FN], f2a[FM], f2b[FN], f3a[FM], f3b[FN];
  // read q (0..7) of sub-step KK's fragments (A stage SA, weight stage SW) into set B
  auto rd1 = [&](auto kkc, auto sac, auto swc, auto bc, int q) {
    constexpr int KK = decltype(kkc)::value, SA = decltype(sac)::value, SW = decltype(swc)::value;
    constexpr int B = decltype(bc)::value;
    constexpr int OA = SA * SB, OB = SW == 2 ? 0 : SW * SB;
    const uint32_t ab = SW == 2 ? adB2[KK] : adB[KK];
#define SPH_W1_READ(FA, FB)                             \
    switch (q) {                                        \
      case 0: w1_read<OA + 0>(FA[0], adA[KK]); break;     \
      case 1: w1_read<OB + 0>(FB[0], ab); break;          \
      case 2: w1_read<OA + 4096>(FA[1], adA[KK]); break;  \
      case 3: w1_read<OB + 4096>(FB[1], ab); break;       \
      case 4: w1_read<OA + 8192>(FA[2], adA[KK]); break;  \
      case 5: w1_read<OB + 8192>(FB[2], ab); break;       \
      case 6: w1_read<OA + 12288>(FA[3], adA[KK]); break; \
      default: w1_read<OB + 12288>(FB[3], ab); break;     \
    }
    if constexpr (B == 0) { SPH_W1_READ(f0a, f0b) }
    else if constexpr (B == 1) { SPH_W1_READ(f1a, f1b) }
    else if constexpr (B == 2) { SPH_W1_READ(f2a, f2b) }
    else { SPH_W1_READ(f3a, f3b) }
#undef SPH_W1_READ
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  // the 16 MFMAs of set B, hook(t) after MFMA t; the set stays allocated to the end
  auto phase = [&](auto bc, auto hook) {
    constexpr int B = decltype(bc)::value;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int i = t >> 2, j = t & 3;
      if constexpr (B == 0) w1_mfma(acc[i][j], f0a[i], f0b[j]);
      else if constexpr (B == 1) w1_mfma(acc[i][j], f1a[i], f1b[j]);
      else if constexpr (B == 2) w1_mfma(acc[i][j], f2a[i], f2b[j]);
      else w1_mfma(acc[i][j], f3a[i], f3b[j]);
      hook(t);
    }
    if constexpr (B == 0)
      asm volatile("" :: "v"(f0a[0]), "v"(f0a[1]), "v"(f0a[2]), "v"(f0a[3]), "v"(f0b[0]), "v"(f0b[1]), "v"(f0b[2]), "v"(f0b[3]));
    else if constexpr (B == 1)
      asm volatile("" :: "v"(f1a[0]), "v"(f1a[1]), "v"(f1a[2]), "v"(f1a[3]), "v"(f1b[0]), "v"(f1b[1]), "v"(f1b[2]), "v"(f1b[3]));
    else if constexpr (B == 2)
      asm volatile("" :: "v"(f2a[0]), "v"(f2a[1]), "v"(f2a[2]), "v"(f2a[3]), "v"(f2b[0]), "v"(f2b[1]), "v"(f2b[2]), "v"(f2b[3]));
    else
      asm volatile("" :: "v"(f3a[0]), "v"(f3a[1]), "v"(f3a[2]), "v"(f3a[3]), "v"(f3b[0]), "v"(f3b[1]), "v"(f3b[2]), "v"(f3b[3]));
  };
  // step s, with h stage SA = s % 2 and weight stage SW = s % NB: the weights
  // for step s + NB and h for step s + 2 are copied into this step's stages
  // after the barrier (past the end: the last step again)
  auto step = [&](auto sac, auto swc, int s) {
    constexpr int SA = decltype(sac)::value, SW = decltype(swc)::value;
    using SAc = std::integral_constant<int, SA>;
    using SWc = std::integral_constant<int, SW>;
    using SAn = std::integral_constant<int, SA ^ 1>;
    using SWn = std::integral_constant<int, (SW + 1) % NB>;
    const int sa = min(s + 2, S - 1), sw = min(s + NB, S - 1);
    // three weight stages: this step's first two sub-steps copy the weights
    // of step s + 2 (4 copies each, one per 4 MFMAs) into the stage step
    // s - 1 read
    constexpr int SWp = (SW + 2) % 3;
    w1_wait_lds8();
    phase(I0{}, [&](int t) {
      if (t < 8) rd1(I2{}, SAc{}, SWc{}, I2{}, t);
      if (NB == 3 && s > 0 && (t & 3) == 1) copyB(t >> 2, sa, SWp);
    });
    w1_wait_lds8();
    phase(I1{}, [&](int t) {
      if (t < 8) rd1(I3{}, SAc{}, SWc{}, I3{}, t);
      if (NB == 3 && s > 0 && (t & 3) == 1) copyB(4 + (t >> 2), sa, SWp);
    });
    // this wave's reads of the stages are done, and its copies for the next
    // step have landed (with three weight stages the newest 8, the weights of
    // step s + 2, may still be in flight)
    w1_wait_lds();
    if constexpr (NB == 2) w1_wait_mem();
    else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if constexpr (NB == 2) {
      phase(I2{}, [&](int t) {
        if (t < 8) {
          rd1(I0{}, SAn{}, SWn{}, I0{}, t);
          copyA(t, sa, SA);
        }
      });
      w1_wait_lds8();
      phase(I3{}, [&](int t) {
        if (t < 8) {
          rd1(I1{}, SAn{}, SWn{}, I1{}, t);
          copyB(t, sw, SW);
        }
      });
    } else {
      // h of step s + 2 into this step's h stage, 4 copies per sub-step
      phase(I2{}, [&](int t) {
        if (t < 8) rd1(I0{}, SAn{}, SWn{}, I0{}, t);
        if ((t & 3) == 1) copyA(t >> 2, sa, SA);
      });
      w1_wait_lds8();
      phase(I3{}, [&](int t) {
        if (t < 8) rd1(I1{}, SAn{}, SWn{}, I1{}, t);
        if ((t & 3) == 1) copyA(4 + (t >> 2), sa, SA);
      });
    }
  };
  // prologue: h steps 0 and 1, weight steps 0 .. NB - 1; steps 0 land first
#pragma unroll
  for (int i = 0; i < A_INS; ++i) copyA(i, 0, 0);
#pragma unroll
  for (int i = 0; i < B_INS; ++i) copyB(i, 0, 0);
#pragma unroll
  for (int i = 0; i < A_INS; ++i) copyA(i, 1, 1);
#pragma unroll
  for (int i = 0; i < B_INS; ++i) copyB(i, 1, 1);
  if constexpr (NB == 3) {
#pragma unroll
    for (int i = 0; i < B_INS; ++i) copyB(i, 2, 2);
    asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 8; ++q) rd1(I0{}, I0{}, I0{}, I0{}, q);
#pragma unroll
  for (int q = 0; q < 8; ++q) rd1(I1{}, I0{}, I0{}, I1{}, q);
  if constexpr (NB == 2) {
    for (int s = 0; s < S; s += 2) {
      step(I0{}, I0{}, s);
      step(I1{}, I1{}, s + 1);
    }
  } else {
    for (int s = 0; s < S; s += 6) {
      step(I0{}, I0{}, s);
      step(I1{}, I1{}, s + 1);
      step(I0{}, I2{}, s + 2);
      step(I1{}, I0{}, s + 3);
      step(I0{}, I1{}, s + 4);
      step(I1{}, I2{}, s + 5);
    }
  }
  // the last copies (into stages nobody reads) and reads land before the
  // LDS is given up; the last MFMAs' results are written before the AGPRs
  // are read
  w1_wait_mem();
  w1_wait_lds();
  // (the sets that the last reads fill stay allocated until those have landed:
  // without this a register of theirs was given to the epilogue before the wait)
  asm volatile("" :: "v"(f0a[0]), "v"(f0a[1]), "v"(f0a[2]), "v"(f0a[3]), "v"(f0b[0]), "v"(f0b[1]), "v"(f0b[2]), "v"(f0b[3]));
  asm volatile("" :: "v"(f1a[0]), "v"(f1a[1]), "v"(f1a[2]), "v"(f1a[3]), "v"(f1b[0]), "v"(f1b[1]), "v"(f1b[2]), "v"(f1b[3]));
  asm volatile("s_nop 7\n s_nop 7\n s_nop 7\n s_nop 7\n s_nop 7\n s_nop 7\n s_nop 7\n s_nop 7" ::: "memory");
  if constexpr (NB == 3) {
    __syncthreads();  // every wave is done with the stages: the row maxima take the first
    for (int i = tid; i < BM; i += NT) s_rmax[i] = 0u;
    __syncthreads();
  }

  // Epilogue: each fragment leaves the AGPRs on its own (the generic tile
  // epilogue, which reads all 256 accumulators, spilled); z and the tile's
  // row maxima of |clamp(z)| as there.
  constexpr int P = FM * 16;
  float red[P];
#pragma unroll
  for (int t = 0; t < P; ++t) red[t] = 0.0f;
  const float clip = a.clip;
  const int ldz = a.ldz;
  const auto rsrc = tile_rsrc(a.z + (int64_t)m0 * ldz, min(BM, M - m0), ldz);
  const uint32_t lrow0 = (uint32_t)(wm * TM + 4 * (lane >> 5));
  const uint32_t lcol0 = (uint32_t)(n0 + wn * TN + (lane & 31));
  auto fill = [&](auto plain) {
    constexpr bool PL = decltype(plain)::value;  // no bias, a tile inside the positions
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        f32x16_t v;
        asm volatile("; fragment out of the AGPRs" : "=v"(v) : "0"(acc[i][j]));
        const uint32_t col = lcol0 + 32u * j;
        uint32_t off = ((lrow0 + 32u * i) * (uint32_t)ldz + col) * 4u;
        float cb = 0.0f;
        if (!PL && a.bias) {
          const int lcol = wn * TN + j * 32 + (lane & 31);
          cb = a.bias[NB == 2 ? s_ids[lcol] : (col < (uint32_t)n ? a.ids[col] : last_id)];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float zv = !PL && a.bias ? v[r] + cb : v[r];
          if (r > 0) next_row(off, r, ldz);
          store_z(zv, rsrc, !PL && col >= (uint32_t)n ? kPastTile : off);
          red[i * 16 + r] = fmaxf(red[i * 16 + r], fminf(fabsf(zv), clip));
        }
      }
    }
  };
  if (n0 + BN <= n && !a.bias) fill(std::true_type{});
  else fill(std::false_type{});
  half_wave_max_transpose<P>(red, lane);
  constexpr int PER = P / 32;
#pragma unroll
  for (int t = 0; t < PER; ++t) {
    const int idx = (lane & 31) * PER + t;
    const int i = idx / 16, r = idx % 16;
    const int lrow = wm * TM + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    atomicMax(&s_rmax[lrow], __float_as_uint(red[t]));
  }
  __syncthreads();
  for (int i = tid; i < BM; i += NT)
    if (m0 + i < M) a.amax_part[(int64_t)(m0 + i) * kMaxBlocks + nt] = __uint_as_float(s_rmax[i]);
#endif
}

// Tiles of fp8 E4M3 weights, K a multiple of 16 (TAIL as above).  The A
// tile is staged as above; the B tile keeps its bytes: a weight row holds 64
// codes per K step (64 bytes, four 16-byte chunks), and a wave instruction
// fills 16 rows.  Chunks are XOR-swizzled with g(row) = (row >> 2) & 3, so
// the 32 rows a fragment read touches spread over the LDS banks.  Each lane
// reads its 8 codes of a fragment (ds_read_b64) and widens them to bf16
// (exact) in registers right before the MFMA; the per-row scale is applied
// in the epilogue.  The step's codes are read first, then the next stage's
// loads go out and each sub-step reads its own fragments of h; the SIMD's
// other wave covers the wait.
__device__ __forceinline__ int swz4(int row) { return (row >> 2) & 3; }

template <int BM, int BN, int WM, int WN, int EPI, bool O32, bool TAIL>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(WM * WN / 4, WM * WN / 4)))
void k_mfma_dma8(const MfmaArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NT = 64 * WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / 32, FN = TN / 32;
  constexpr int IW = WM * WN / 2;  // as in k_mfma_dma
  constexpr int A_INS = BM / 8 / IW, B_INS = BN / 16 / IW;  // copy instructions per issuing wave per step
  static_assert(A_INS * 8 * IW == BM && B_INS * 16 * IW == BN, "tile rows / issuing waves");
  extern __shared__ __align__(16) uint8_t smem[];
  uint16_t* As = reinterpret_cast<uint16_t*>(smem);             // [2][BM][64] bf16
  uint8_t* Bs = reinterpret_cast<uint8_t*>(As + 2 * BM * kBK);   // [2][BN][64] fp8
  int32_t* s_ids = reinterpret_cast<int32_t*>(Bs + 2 * BN * kBK);
  uint32_t* s_rmax = reinterpret_cast<uint32_t*>(s_ids + BN);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int iw = wave < IW ? wave : 0;  // issuing slot (waves >= IW issue nothing)
  const int wm = wave / WN, wn = wave % WN;
  int mt, nt;
  tile_of_block(blockIdx.x, a.m_tiles, a.n_tiles, mt, nt);
  const int m0 = mt * BM, n0 = nt * BN;
  const int M = a.M, K = a.K, n = a.n;
  const int last_id = a.ids[min(n, n0 + BN) - 1];
  for (int i = tid; i < BN; i += NT) s_ids[i] = n0 + i < n ? a.ids[n0 + i] : last_id;
  for (int i = tid; i < BM; i += NT) s_rmax[i] = 0u;
  __syncthreads();

  const uint8_t* hbase = reinterpret_cast<const uint8_t*>(a.h);
  LaneAddr<O32> pa[A_INS], pb[B_INS];
#pragma unroll
  for (int i = 0; i < A_INS; ++i) {
    const int r = (iw * A_INS + i) * 8 + (lane >> 3);
    const int lc = (lane & 7) ^ swz8(r);
    pa[i].set(hbase, (int64_t)min(m0 + r, M - 1) * a.ldh * 2 + lc * 16);
  }
#pragma unroll
  for (int i = 0; i < B_INS; ++i) {
    const int r = (iw * B_INS + i) * 16 + (lane >> 2);
    const int lc = (lane & 3) ^ swz4(r);
    pb[i].set(a.w, (int64_t)s_ids[r] * a.ldw_bytes + lc * 16);
  }
  auto issue = [&](int k0, int stage) {
    if (wave >= IW) return;
    uint8_t* as = reinterpret_cast<uint8_t*>(As + stage * BM * kBK);
    uint8_t* bs = Bs + stage * BN * kBK;
    const uint8_t* ha = O32 ? scalar_ptr(hbase + (int64_t)k0 * 2) : nullptr;
    const uint8_t* wb = O32 ? scalar_ptr(a.w + k0) : nullptr;
    if (!TAIL || K - k0 >= kBK) {
#pragma unroll
      for (int i = 0; i < A_INS; ++i)
        pa[i].copy(ha, (int64_t)k0 * 2, (lds_void_t*)(as + (iw * A_INS + i) * 1024));
#pragma unroll
      for (int i = 0; i < B_INS; ++i) pb[i].copy(wb, k0, (lds_void_t*)(bs + (iw * B_INS + i) * 1024));
    } else {
      const int valid = K - k0;
#pragma unroll
      for (int i = 0; i < A_INS; ++i) {
        const int c = (lane & 7) ^ swz8((iw * A_INS + i) * 8 + (lane >> 3));
        pa[i].copy_back(ha, (int64_t)k0 * 2, (lds_void_t*)(as + (iw * A_INS + i) * 1024),
                        c * 8 < valid ? 0u : (uint32_t)(c * 16));
      }
#pragma unroll
      for (int i = 0; i < B_INS; ++i) {
        const int c = (lane & 3) ^ swz4((iw * B_INS + i) * 16 + (lane >> 2));
        pb[i].copy_back(wb, k0, (lds_void_t*)(bs + (iw * B_INS + i) * 1024),
                        c * 16 < valid ? 0u : (uint32_t)(c * 16));
      }
    }
  };

  f32x16_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  if (K > 0) {
    issue(0, 0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }
  int stage = 0;
  for (int k0 = 0; k0 < K; k0 += kBK) {
    const uint16_t* as = As + stage * BM * kBK;
    const uint8_t* bs = Bs + stage * BN * kBK;
    if (TAIL && K - k0 < kBK) {
      const int valid = K - k0;
      zero_tail<BM, NT>(As + stage * BM * kBK, valid);
      for (int i = tid; i < BN * 4; i += NT) {
        const int row = i >> 2, c = i & 3;
        if (c * 16 >= valid)
          *reinterpret_cast<u32x4_t*>(Bs + stage * BN * kBK + row * kBK + ((c ^ swz4(row)) << 4)) =
              u32x4_t{0u, 0u, 0u, 0u};
      }
      __syncthreads();
    }
    // The step's fp8 codes (8 bytes per fragment and sub-step, 16 VGPRs)
    // are read before the next stage's copies go out.  The compiler makes
    // an LDS read behind pending copies wait for them where it cannot
    // tell the two apart, and it did so for these 8-byte reads: placed
    // after the copies, they held the issuing wave of each SIMD until its
    // copies had landed, every step (sample_fp8 cloud 438 against 365 us).
    uint2 qb[kBK / 16][FN];
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int row = wn * TN + j * 32 + (lane & 31);
        qb[kk][j] = *reinterpret_cast<const uint2*>(bs + row * kBK + ((kk ^ swz4(row)) << 4) + 8 * (lane >> 5));
      }
    if (k0 + kBK < K) issue(k0 + kBK, stage ^ 1);
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      const int c = kk * 2 + (lane >> 5);
      bf16x8_t af[FM], bfr[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int row = wm * TM + i * 32 + (lane & 31);
        af[i] = *reinterpret_cast<const bf16x8_t*>(as + row * kBK + ((c ^ swz8(row)) << 3));
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const uint2 q = qb[kk][j];
        u32x4_t w;
        w.x = e4m3x2_to_bf16x2_m<false>(q.x);
        w.y = e4m3x2_to_bf16x2_m<true>(q.x);
        w.z = e4m3x2_to_bf16x2_m<false>(q.y);
        w.w = e4m3x2_to_bf16x2_m<true>(q.y);
        bfr[j] = __builtin_bit_cast(bf16x8_t, w);
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    stage ^= 1;
  }
  tile_epilogue<BM, BN, WM, WN, 1, EPI>(acc, a, s_ids, s_rmax, m0, n0, nt, reinterpret_cast<int8_t*>(As));
#endif
}

template <int BM, int BN>
constexpr size_t mfma_dma_lds_bytes() {
  return (size_t)2 * (BM + BN) * kBK * 2 + (size_t)BN * 4 + (size_t)BM * 4;
}

template <int BM, int BN>
constexpr size_t mfma_dma8_lds_bytes() {
  return (size_t)2 * (BM * 2 + BN) * kBK + (size_t)BN * 4 + (size_t)BM * 4;
}

// Waves of a cloud row tile (the direct-to-LDS kernels): 8, two per SIMD, so
// one wave's MFMAs run while the other waits at a barrier or on LDS: 2 x 4
// (wave tiles 128 x 64 / 160 x 64), whose long K loop ran 6% faster so than
// with 4 x 2; on the dense 2048-row shape 8 waves ran 9% faster than 4 (wave
// tile 128 x 128).
constexpr int kTileWM = 2, kTileWN = 4;

template <int BM, int BN, int WT, int EPI, bool O32, bool TAIL>
static hipError_t launch_dma(const MfmaArgs& a, hipStream_t s) {
  static std::atomic<uint64_t> lds_set{0};
  constexpr int WM = kTileWM, WN = kTileWN;
  auto k = [] {
    if constexpr (WT == 0) return k_mfma_dma<BM, BN, WM, WN, EPI, O32, TAIL>;
    else return k_mfma_dma8<BM, BN, WM, WN, EPI, O32, TAIL>;
  }();
  constexpr size_t lds = WT == 0 ? mfma_dma_lds_bytes<BM, BN>() : mfma_dma8_lds_bytes<BM, BN>();
  hipError_t e = set_lds_limit_once(lds_set, reinterpret_cast<const void*>(k), lds);
  if (e != hipSuccess) return e;
  launch_kernel(k, dim3(a.m_tiles * a.n_tiles), dim3(64 * WM * WN), lds, s, a);
  return hipGetLastError();
}

template <int NB>
static hipError_t launch_w1(const MfmaArgs& a, size_t lds, hipStream_t s) {
  static std::atomic<uint64_t> lds_set{0};
  auto k = k_mfma_w1<kEpiCloud, NB>;
  hipError_t e = set_lds_limit_once(lds_set, reinterpret_cast<const void*>(k), lds);
  if (e != hipSuccess) return e;
  launch_kernel(k, dim3(a.m_tiles * a.n_tiles), dim3(256), lds, s, a);
  return hipGetLastError();
}

// (the one-wave kernels copy their first steps unconditionally: they need at
// least 6 or 2 steps; fewer take the two-wave kernel)
int mfma_w1_stages(int K) {
  if (K % kBK != 0 || K < 2 * kBK) return 0;
  const int steps = K / kBK;
  return steps % 6 == 0 ? 3 : steps % 2 == 0 ? 2 : 0;
}

template <int BM, int BN, int WT, int EPI>
static hipError_t launch_tile(MfmaArgs a, hipStream_t s) {
  a.m_tiles = (a.M + BM - 1) / BM;
  a.n_tiles = (a.n + BN - 1) / BN;
  if (a.n_tiles > kMaxBlocks || a.K % (WT == 0 ? 8 : 16) != 0) return hipErrorInvalidValue;
  const bool o32 = copy_offsets_fit(a), tail = a.K % kBK != 0;
  if constexpr (BM == 256 && WT == 0 && EPI == kEpiCloud) {
    const int stages = o32 ? mfma_w1_stages(a.K) : 0;
    if (stages == 3) return launch_w1<3>(a, (size_t)5 * BM * kBK * 2, s);  // all 160 KB of LDS
    if (stages == 2) return launch_w1<2>(a, mfma_dma_lds_bytes<BM, BN>(), s);
  }
  if (o32)
    return tail ? launch_dma<BM, BN, WT, EPI, true, true>(a, s) : launch_dma<BM, BN, WT, EPI, true, false>(a, s);
  return tail ? launch_dma<BM, BN, WT, EPI, false, true>(a, s) : launch_dma<BM, BN, WT, EPI, false, false>(a, s);
}

// Row tile for M rows (more than kStreamMaxRows): whichever of 256 and 320
// pads M less.  Measured on
// the batched shape (M = 320, 60000 ids): 320-row tiles, one per 256 ids,
// 156 us against 265 us for 256-row tiles; M = 640 with fp8 weights: 460 us
// against 537 us for 256-row tiles.
int mfma_bm(int M) {
  const int pad256 = (M + 255) / 256 * 256 - M;
  const int pad320 = (M + 319) / 320 * 320 - M;
  return pad320 < pad256 ? 320 : 256;
}

int mfma_n_tiles(int n) { return (n + kMfmaBN - 1) / kMfmaBN; }
int mfma_tiles(int M, int n) { return (M + mfma_bm(M) - 1) / mfma_bm(M) * mfma_n_tiles(n); }

template <int WT, int EPI>
static hipError_t launch_bm(const MfmaArgs& a, hipStream_t s) {
  return mfma_bm(a.M) == 320 ? launch_tile<320, kMfmaBN, WT, EPI>(a, s)
                                  : launch_tile<256, kMfmaBN, WT, EPI>(a, s);
}

// Cloud projection with the block quantiser in the epilogue, for the row
// tile whose accumulators and row maxima fit in the registers together
// (256 rows).  Where the tile rule picks 320 rows the separate quantiser is
// used: on 640 rows, 256-row tiles with the fused quantiser ran 598 us against
// 428 + 43 us.
// With a partial last K step only where there are four rounds of tiles or more
// (a tile's quantising epilogue keeps its CU some 30 us, the separate one
// shares out evenly), and for E4M3 weights, whose steps hide less of it, only
// for long K and code rows that start on 128-byte lines.  (us, in the epilogue /
// separate, bf16: 1964 rows x 863 positions x 208 columns 45 / 21, 512 x 100000 x
// 1008 243 / 224, 1200 x 60000 x 1008 291 / 279, 2048 x 32768 x 1008 240 / 265,
// 1024 x 128256 x 4016 1248 / 1300; E4M3: 2048 x 32768 x 1008 264 / 257, x 4016
// 572 / 590, 2048 x 60000 x 208 353 / 291, x 4016 1105 / 1073.)
bool mfma_quantises_in_epilogue(int M, int n, int K, int wtype, int bits) {
  if (mfma_bm(M) == 320) return false;
  if (K % kBK == 0) return true;
  if (mfma_tiles(M, n) < 4 * kCUs) return false;
  return wtype == 0 || (K >= 2048 && (int64_t)n * bits % (128 * 8) == 0);
}

template <int WT>
static hipError_t launch_bm_q(const MfmaArgs& a, hipStream_t s) {
  if (!mfma_quantises_in_epilogue(a.M, a.n, a.K, WT, a.qout_bits)) return hipErrorInvalidValue;
  return launch_tile<256, kMfmaBN, WT, kEpiCloudQ>(a, s);
}

hipError_t launch_mfma(int epi, int wtype, const MfmaArgs& a, hipStream_t s) {
  if (epi == kEpiCloudQ) return wtype == 0 ? launch_bm_q<0>(a, s) : launch_bm_q<1>(a, s);
  if (epi == kEpiCloud)
    return wtype == 0 ? launch_bm<0, kEpiCloud>(a, s) : launch_bm<1, kEpiCloud>(a, s);
  return wtype == 0 ? launch_fuse_mfma(a, s) : hipErrorInvalidValue;
}

}  // namespace sph
