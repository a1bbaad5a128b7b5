// Endpoint projection of many rows of h on the matrix cores (eqs. 11, 13-14).
#include "mfma_tile.h"

namespace sph {

// 16 payload bytes at p, of which the first `left` (at least 1) belong to the
// row; bytes past it are 0.  p may have any alignment (an unaligned 16-byte
// load is one instruction).
__device__ __forceinline__ u32x4_t load_chunk16(const uint8_t* p, int64_t left) {
  u32x4_t v = {0u, 0u, 0u, 0u};
  if (left >= 16) {
    __builtin_memcpy(&v, p, 16);
  } else {
    uint64_t lo = 0, hi = 0;
#pragma unroll 1
    for (int b = 0; b < (int)left; ++b) {
      const uint64_t x = p[b];
      if (b < 8) lo |= x << (8 * b);
      else hi |= x << (8 * (b - 8));
    }
    v = u32x4_t{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
  }
  return v;
}

// Endpoint projection with its fuse epilogue (eqs. 11, 13-14), K a multiple
// of 8 (TAIL: the last K step is partial and its missing columns are zeroed in
// LDS; a second loop body with fewer sub-steps doubled the accumulators).
// The block computes the transposed tile C^T[n][m] =
// W[S_n] . h[m]: the weight rows are the MFMA's A operand and the rows of h
// its B operand.  The weight rows of each 32-row group are staged in the
// order that puts subset position 16*(l/32) + r of the group in accumulator
// r of lane l: a lane holds 16 consecutive positions of row j*32 + l%32 (in
// the wave's tile) per fragment.  Operands are otherwise staged exactly as
// in k_mfma_dma.  A BM x BN tile runs WNN x WMM waves (WNN along the
// positions, WMM along the rows).
//
// Payload: the tile's codes (BM rows of BN * qbits / 8 bytes) are staged
// in LDS as 16-byte chunks, swizzled per row, so one 16-byte read gives a
// lane its 16 8-bit codes (an 8-byte read its 16 4-bit codes) and the rows
// a read touches spread over the banks.  With 8-bit codes on 16-byte
// aligned rows the tile is copied global-to-LDS during the last K step into
// the operand buffers that step does not read (rows [0, BM/2) into the idle
// A buffer, the rest into the idle B buffer), where it lands while the last
// MFMAs run; otherwise it passes through registers (load_payload).
//
// Selection: f = fma(code, s, dot * hs) (the product only with hidden-state
// scales), the lane's largest f, then the lowest of the lane's positions
// holding it; the two lanes holding a row (l, l ^ 32) keep the larger
// orderable key (value, then lowest position), and LDS atomics combine the
// WNN waves sharing the row.  Against the row-major epilogue (one LDS byte
// read per code and a 32-lane butterfly of 64-bit keys) the first form of
// this kernel (four positions per register group, a 32-bit code read and a
// running compare per value) ran dense_full's endpoint projection in 358 us
// instead of 505, dense_sub in 85 instead of 114 and batched in 29 instead
// of 47; the 16-position layout then took dense_sub to 81 us and batched to
// 27, with identical keys throughout.  One wave per SIMD instead (the cloud
// kernel's explicit schedule with 128 x 128 wave tiles, the payload copied in
// place of the copies past the end) kept the keys identical but ran slower:
// with 8 K steps a tile's prologue and epilogue weigh more than the LDS
// traffic the larger wave tiles save (dense_full 379-396 against 350-364 us,
// dense_sub 87 against 76).
template <int BM, int BN>
constexpr size_t fuse_dma_lds_bytes() {
  return (size_t)2 * (BM + BN) * kBK * 2 + (size_t)BN * 4 + (size_t)2 * BM * 4 + (size_t)BM * 8;
}

template <int BM, int BN, int WNN, int WMM, int BPC, bool O32, bool TAIL>
__global__ __launch_bounds__(64 * WNN * WMM)
__attribute__((amdgpu_waves_per_eu(WNN * WMM / 4 * BPC, WNN * WMM / 4 * BPC)))
void k_fuse_dma(const MfmaArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NT = 64 * WNN * WMM;
  constexpr int FI = BN / WNN / 32, FJ = BM / WMM / 32;  // position / row fragments per wave
  static_assert(FI * WNN * 32 == BN && FJ * WMM * 32 == BM, "wave grid");
  constexpr int IW = 4;  // waves issuing the operand copies (one per SIMD)
  constexpr int A_INS = BM / 8 / IW, B_INS = BN / 8 / IW;
  static_assert(A_INS * 8 * IW == BM && B_INS * 8 * IW == BN, "copy instructions");
  constexpr int STAGE_B = (BM + BN) * kBK * 2;  // bytes of one operand stage
  constexpr bool kLastStep = BM <= 256;  // an 8-bit tile's halves fit the two buffers of a stage
  extern __shared__ __align__(16) uint8_t smem[];
  uint16_t* As = reinterpret_cast<uint16_t*>(smem);                 // [2][BM][64]
  uint16_t* Bs = As + 2 * BM * kBK;                                  // [2][BN][64]
  int32_t* s_ids = reinterpret_cast<int32_t*>(smem + 2 * STAGE_B);
  float* s_sc = reinterpret_cast<float*>(s_ids + BN);               // [2][BM]: scale, dot factor
  unsigned long long* s_rkey = reinterpret_cast<unsigned long long*>(s_sc + 2 * BM);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int iw = wave < IW ? wave : 0;
  const int wn = wave % WNN, wm = wave / WNN;
  int mt, nt;
  tile_of_block(blockIdx.x, a.m_tiles, a.n_tiles, mt, nt);
  const int m0 = mt * BM, n0 = nt * BN;
  const int M = a.M, K = a.K, n = a.n;
  const int last_id = a.ids[min(n, n0 + BN) - 1];
  for (int i = tid; i < BN; i += NT) s_ids[i] = n0 + i < n ? a.ids[n0 + i] : last_id;
  // a tile lies in one block of positions (blocks are multiples of BN)
  const int kb = a.qshift < 0 ? 0 : (n0 >> a.qshift);
  for (int i = tid; i < BM; i += NT) {
    s_rkey[i] = 0ull;
    s_sc[i] = m0 + i < M ? a.qscale[(int64_t)(m0 + i) * a.qnb + kb] : 0.0f;
    s_sc[BM + i] = (a.hscale && m0 + i < M) ? a.hscale[m0 + i] : 1.0f;
  }
  __syncthreads();
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
    // weight row r of a 32-row group holds subset position pr: MFMA row
    // 8g + 4h + e (g = register group, h = lane / 32, e = element) gets
    // position 16h + 4g + e, so a lane's 16 accumulators cover 16
    // consecutive positions
    const int pr = (r & ~31) | (((r >> 2) & 1) << 4) | (((r >> 3) & 3) << 2) | (r & 3);
    pb[i].set(a.w, (int64_t)s_ids[pr] * a.ldw_bytes + lc * 16);
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
      // the last, partial step: chunks at or past K read the step's first
      // chunk instead (in bounds; zero_tail clears them)
      const uint32_t valid = (uint32_t)(K - k0) * 2;
      auto back = [&](int r) {
        const uint32_t c = (uint32_t)((lane & 7) ^ swz8(r)) * 16u;
        return c < valid ? 0u : c;
      };
#pragma unroll
      for (int i = 0; i < A_INS; ++i)
        pa[i].copy_back(ha, step, (lds_void_t*)(as + (iw * A_INS + i) * 1024), back((iw * A_INS + i) * 8 + lr));
#pragma unroll
      for (int i = 0; i < B_INS; ++i)
        pb[i].copy_back(wb, step, (lds_void_t*)(bs + (iw * B_INS + i) * 1024), back((iw * B_INS + i) * 8 + lr));
    }
  };
  const int qb = a.qbits;
  const int TB = BN * qb / 8;  // code bytes of a tile row
  const int CPR = TB / 16;     // 16-byte chunks of a tile row
  const int64_t c0 = (int64_t)n0 * qb / 8;
  const int64_t rowbytes = ((int64_t)n * qb + 7) / 8;
  const bool vec_q = (a.qstride & 15) == 0 && (reinterpret_cast<uintptr_t>(a.q) & 15) == 0;
  const bool dma_q = qb == 8 && vec_q;
  // chunk swizzle of payload row r: 16 (BN = 256) or 8 chunks of 8-bit codes, 8
  // or 4 of 4-bit codes (by r / 2 or r / 4, so that the 8-byte reads of 32 rows
  // spread over the banks)
  auto qswz8 = [](int r) { return BN == 256 ? (r & 15) : swz8(r); };
  auto qswz4 = [](int r) { return BN == 256 ? ((r >> 1) & 7) : ((r >> 2) & 3); };
  auto qswz = [&](int r) { return qb == 8 ? qswz8(r) : qswz4(r); };
  // payload row r: staged in the last K step, rows [0, BM/2) in the idle
  // stage's A buffer and [BM/2, BM) in its B buffer; staged after the
  // loop, consecutive rows from the start of LDS
  auto prow = [&](bool in_stage, int st, int r) -> uint8_t* {
    if (!in_stage) return smem + r * TB;
    return r < BM / 2 ? reinterpret_cast<uint8_t*>(As + st * BM * kBK) + r * TB
                      : reinterpret_cast<uint8_t*>(Bs + st * BN * kBK) + (r - BM / 2) * TB;
  };
  // global-to-LDS copies of an 8-bit payload tile: a wave instruction fills
  // 1 KB (RP rows, contiguous in either placement); rows past M read row
  // M-1 and chunks past the row's end read the tile's first chunk (their
  // positions are never selected)
  auto stage_payload_dma = [&](bool in_stage, int st) {
    constexpr int RP = 1024 / BN, CP = BN / 16;
    for (int t = wave; t < BM / RP; t += WNN * WMM) {
      const int r = t * RP + lane / CP;
      const int k = (lane & (CP - 1)) ^ qswz8(r);
      const int64_t col = c0 + k * 16 < rowbytes ? c0 + k * 16 : c0;
      __builtin_amdgcn_global_load_lds(a.q + (int64_t)min(m0 + r, M - 1) * a.qstride + col,
                                       (lds_void_t*)prow(in_stage, st, t * RP), 16, 0, 0);
    }
  };

  // Every other payload tile (4-bit codes, or rows that are not 16-byte
  // aligned: any 8-bit row of a subset whose size is no multiple of 16)
  // passes through registers after the loop, 16 bytes per load at whatever
  // alignment the row has and all of a thread's loads in flight at once.
  // (Byte loads took 30 us of a launch: 18 rows x 45001 ids 29.7 -> 8.3 us
  // together with the partial K step below, 78 x 36974 51.4 -> 27.3.  Loading
  // before the last step's MFMAs spilled the accumulators of two waves per
  // SIMD and gained nothing with one.)
  constexpr int QT = BM * (BN / 16) / NT;  // 8-bit chunks per thread (4-bit: half of them)
  u32x4_t qv[QT];
  auto load_payload = [&]() {
    const int ksh = (BN == 256 ? 4 : 3) - (qb == 8 ? 0 : 1);  // log2 CPR
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      const int c = tid + t * NT, r = c >> ksh;
      const int64_t col = c0 + (int64_t)(c & (CPR - 1)) * 16;
      qv[t] = u32x4_t{0u, 0u, 0u, 0u};
      if (r < BM && m0 + r < M && col < rowbytes)
        qv[t] = load_chunk16(a.q + (int64_t)(m0 + r) * a.qstride + col, rowbytes - col);
    }
  };
  auto store_payload = [&]() {
    const int ksh = (BN == 256 ? 4 : 3) - (qb == 8 ? 0 : 1);
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      const int c = tid + t * NT, r = c >> ksh, k = c & (CPR - 1);
      if (r < BM) *reinterpret_cast<u32x4_t*>(smem + r * TB + ((k ^ qswz(r)) << 4)) = qv[t];
    }
  };

  f32x16_t acc[FI][FJ];
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < FJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  if (K > 0) {
    issue(0, 0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }
  int stage = 0;
  bool staged = false;
  for (int k0 = 0; k0 < K; k0 += kBK) {
    if (k0 + kBK < K) {
      issue(k0 + kBK, stage ^ 1);
    } else if (kLastStep && dma_q) {
      // the last step reads one stage; the payload tile goes to the other
      stage_payload_dma(true, stage ^ 1);
      staged = true;
    }
    const uint16_t* as = As + stage * BM * kBK;
    const uint16_t* bs = Bs + stage * BN * kBK;
    if (TAIL && K - k0 < kBK) {
      zero_tail<BM, NT>(As + stage * BM * kBK, K - k0);
      zero_tail<BN, NT>(Bs + stage * BN * kBK, K - k0);
      __syncthreads();
    }
#pragma unroll
    for (int kk = 0; kk < kBK / 16; ++kk) {
      bf16x8_t hf[FJ], wf[FI];
      const int c = kk * 2 + (lane >> 5);
#pragma unroll
      for (int j = 0; j < FJ; ++j) {
        const int row = wm * (BM / WMM) + j * 32 + (lane & 31);
        hf[j] = *reinterpret_cast<const bf16x8_t*>(as + row * kBK + ((c ^ swz8(row)) << 3));
      }
#pragma unroll
      for (int i = 0; i < FI; ++i) {
        const int row = wn * (BN / WNN) + i * 32 + (lane & 31);
        wf[i] = *reinterpret_cast<const bf16x8_t*>(bs + row * kBK + ((c ^ swz8(row)) << 3));
      }
#pragma unroll
      for (int i = 0; i < FI; ++i)
#pragma unroll
        for (int j = 0; j < FJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i], hf[j], acc[i][j], 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0);  // this wave's copies (operands or payload) have landed
    __syncthreads();
    stage ^= 1;
  }
  // after the last step's toggle, `stage` names the buffer that step did not read
  const int pst = stage;
  if (!staged) {
    if (dma_q) {
      stage_payload_dma(false, 0);
      __builtin_amdgcn_s_waitcnt(0);
    } else {
      load_payload();
      store_payload();
    }
    __syncthreads();
  }
  // lane l of fragment (i, j) holds positions i*32 + 16*(l/32) + r of row
  // j*32 + l%32 in its 16 accumulators r: one 16-byte (8-bit) or 8-byte
  // (4-bit) LDS read gives the lane its codes; the lane's largest fused
  // value, then the lowest of its positions holding it
  const bool hq = a.hscale != nullptr;
  const int hh = lane >> 5;
  auto run = [&](auto edge, auto hidden) {
    constexpr bool kEdge = decltype(edge)::value;  // bounds checks and the fused output
    constexpr bool kHq = decltype(hidden)::value;  // rows carry hidden-state scales
#pragma unroll
    for (int j = 0; j < FJ; ++j) {
      const int ml = wm * (BM / WMM) + j * 32 + (lane & 31);
      const float sc = s_sc[ml];
      const uint8_t* qrow = prow(staged, pst, ml);
      u32x4_t cq[FI];
#pragma unroll
      for (int i = 0; i < FI; ++i) {
        const int nl0 = wn * (BN / WNN) + i * 32 + 16 * hh;
        if (qb == 8) {
          cq[i] = *reinterpret_cast<const u32x4_t*>(qrow + (((nl0 >> 4) ^ qswz8(ml)) << 4));
        } else {
          const int bo = nl0 >> 1;
          const uint2 h2 = *reinterpret_cast<const uint2*>(qrow + ((((bo >> 4) ^ qswz4(ml)) << 4) | (bo & 15)));
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const uint32_t h = ((g < 2 ? h2.x : h2.y) >> (16 * (g & 1))) & 0xFFFFu;
            uint32_t c4 = (h & 0xFu) | ((h & 0xF0u) << 4) | ((h & 0xF00u) << 8) | ((h & 0xF000u) << 12);
            c4 |= (c4 & 0x08080808u) * 0x1Eu;  // a nibble's sign bit fills bits 4..7 of its byte
            cq[i][g] = c4;
          }
        }
      }
      if constexpr (kHq) {
        const float hsc = s_sc[BM + ml];
#pragma unroll
        for (int i = 0; i < FI; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] *= hsc;
      }
      float bv = -__builtin_inff();
#pragma unroll
      for (int i = 0; i < FI; ++i) {
        const int nl0 = wn * (BN / WNN) + i * 32 + 16 * hh;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int code = (int)(int8_t)(cq[i][r >> 2] >> (8 * (r & 3)));
          acc[i][j][r] = __builtin_fmaf((float)code, sc, acc[i][j][r]);
        }
        if constexpr (kEdge) {
          if (a.f) {
            // lanes l and l + 32 trade halves so that each holds positions
            // 8q + 4*(l/32) + [0, 4) in registers 4*ro(q), ro = 0, 2, 1, 3:
            // each store instruction then covers 32 contiguous bytes of a row
            float x[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = acc[i][j][r];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
#pragma unroll
              for (int b = 0; b < 16; b += 8) {
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[b + e]),
                                                                 __float_as_uint(x[b + 4 + e]), false, false);
                x[b + e] = __uint_as_float(sw[0]);
                x[b + 4 + e] = __uint_as_float(sw[1]);
              }
            }
            const int m = m0 + ml;
            if (m < M) {
              const int nlb = wn * (BN / WNN) + i * 32 + 4 * hh;
              float* dst = a.f + (int64_t)m * n + n0 + nlb;
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const int ro = ((q & 1) << 3) | ((q >> 1) << 2);
                if (n0 + nlb + 8 * q + 4 <= n) {  // one store at any alignment
                  const float4 v = make_float4(x[ro], x[ro + 1], x[ro + 2], x[ro + 3]);
                  __builtin_memcpy(dst + 8 * q, &v, 16);
                } else {
#pragma unroll
                  for (int e = 0; e < 4; ++e)
                    if (n0 + nlb + 8 * q + e < n) dst[8 * q + e] = x[ro + e];
                }
              }
            }
          }
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (n0 + nl0 + r >= n) acc[i][j][r] = -__builtin_inff();
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) bv = fmaxf(bv, acc[i][j][r]);
      }
      int bn = 0;
#pragma unroll
      for (int t = FI * 16 - 1; t >= 0; --t) bn = acc[t >> 4][j][t & 15] == bv ? t : bn;
      const int pos = wn * (BN / WNN) + (bn >> 4) * 32 + 16 * hh + (bn & 15);
      unsigned long long key = bv > -__builtin_inff() ? argmax_key_m(bv, n0 + pos) : 0ull;
      const unsigned long long other = xor_lane_u64_32(key);
      key = key > other ? key : other;
      if (lane < 32) atomicMax(&s_rkey[ml], key);
    }
  };
  if (a.f || m0 + BM > M || n0 + BN > n) {
    if (hq) run(std::true_type{}, std::true_type{});
    else run(std::true_type{}, std::false_type{});
  } else {
    if (hq) run(std::false_type{}, std::true_type{});
    else run(std::false_type{}, std::false_type{});
  }
  __syncthreads();
  for (int i = tid; i < BM; i += NT)
    if (m0 + i < M) a.best_part[(int64_t)(m0 + i) * kMaxBlocks + nt] = s_rkey[i];
#endif
}

template <int BM, int BN, int WNN, int WMM, int BPC>
static hipError_t launch_fuse_tile(MfmaArgs a, hipStream_t s) {
  static std::atomic<uint64_t> lds_set[4];
  a.m_tiles = (a.M + BM - 1) / BM;
  a.n_tiles = (a.n + BN - 1) / BN;
  if (a.n_tiles > kMaxBlocks || a.K % 8 != 0) return hipErrorInvalidValue;
  const bool o32 = copy_offsets_fit(a);
  const bool tail = a.K % kBK != 0;
  auto kf = o32 ? (tail ? k_fuse_dma<BM, BN, WNN, WMM, BPC, true, true> : k_fuse_dma<BM, BN, WNN, WMM, BPC, true, false>)
                : (tail ? k_fuse_dma<BM, BN, WNN, WMM, BPC, false, true> : k_fuse_dma<BM, BN, WNN, WMM, BPC, false, false>);
  constexpr size_t lds = fuse_dma_lds_bytes<BM, BN>();
  hipError_t e = set_lds_limit_once(lds_set[2 * o32 + tail], reinterpret_cast<const void*>(kf), lds);
  if (e != hipSuccess) return e;
  launch_kernel(kf, dim3(a.m_tiles * a.n_tiles), dim3(64 * WNN * WMM), lds, s, a);
  return hipGetLastError();
}

// Tiles of 64 (32 up to 32 rows) x 128, three blocks on a CU, or of 256 or 320
// rows (whichever pads M less) x 256, one block.  With few K steps a block is
// mostly waits (ids, first copies, payload), which only other blocks on its CU
// can cover; the large tiles copy less per product.  The small ones up to 128
// rows; where the large ones would leave half of the CUs or more without work;
// and up to 192 rows for short K.  (us, before / small: 18 rows x 45001
// positions x 96 columns 9.2 / 8.2, 60 x 60000 x 512 21.8 / 15.0, 80 x 78720 x
// 512 39 / 29, 128 x 30000 x 256 13.2 / 8.7, 155 x 60000 x 96 15.6 / 13.5, 205 x
// 28982 x 256 4-bit 25 / 16, 320 x 15000 x 512 40 / 15; not taken: 155 x 60000 x
// 512 26.2 / 27.9, 320 x 60000 x 96 17 / 21, x 512 28 / 41, 882 x 29504 x 512
// 50.6 / 50.8, 2048 x 8000 x 512 24 / 27.)
static int fuse_bm_large(int M) { return (M + 319) / 320 * 320 < (M + 255) / 256 * 256 ? 320 : 256; }

static bool fuse_small_tiles(int M, int n, int K) {
  if ((n + 127) / 128 > kMaxBlocks) return false;
  const int bm = fuse_bm_large(M);
  return M <= 128 || (M <= 192 && K <= 256) || (int64_t)((M + bm - 1) / bm) * ((n + 255) / 256) <= kCUs / 2;
}

int fuse_n_tiles(int M, int n, int K) { return fuse_small_tiles(M, n, K) ? (n + 127) / 128 : (n + 255) / 256; }

hipError_t launch_fuse_mfma(const MfmaArgs& a, hipStream_t s) {
  if (fuse_small_tiles(a.M, a.n, a.K))
    return a.M <= 32 ? launch_fuse_tile<32, 128, 4, 1, 3>(a, s) : launch_fuse_tile<64, 128, 4, 1, 3>(a, s);
  // More than 262144 positions, for which the small tiles have no slots.  (us, 64 x
  // 256 / 256 x 256 tiles: 10 rows x 262145 positions x 256 columns 40 / 65, 60 x
  // 300001 x 96 37 / 64, 64 x 400000 x 512 101 / 150, 100 x 262145 x 96 55 / 63;
  // about even past 64 rows with long K: 128 x 300001 x 512 130 / 120.)
  if (a.M <= 128) return launch_fuse_tile<64, 256, 4, 1, 2>(a, s);
  return fuse_bm_large(a.M) == 320 ? launch_fuse_tile<320, 256, 4, 2, 1>(a, s)
                                   : launch_fuse_tile<256, 256, 2, 4, 1>(a, s);
}

}  // namespace sph
