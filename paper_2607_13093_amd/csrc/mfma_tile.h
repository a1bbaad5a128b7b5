// Device helpers shared by the MFMA projection kernels (cloud: mfma.hip,
// endpoint: fuse.hip).
#pragma once

#include <atomic>
#include <type_traits>

#include "sph_internal.h"

namespace sph {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

template <bool HI>
__device__ __forceinline__ uint32_t e4m3x2_to_bf16x2_m(uint32_t x) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(x, 1.0f, HI));
}

__device__ __forceinline__ unsigned long long argmax_key_m(float v, int pos) {
  v = v + 0.0f;  // -0 -> +0
  uint32_t u = __float_as_uint(v);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((unsigned long long)u << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)pos);
}

// z of one accumulator (eq. 12): E4M3 row scale and bias in one rounding, the same
// wherever it is computed (the quantising epilogue computes it twice, and a code
// belongs to the z that its scale came from).
template <int WT>
__device__ __forceinline__ float cloud_value(float dot, float scale, bool has_bias, float bias) {
  if constexpr (WT == 1) return has_bias ? __builtin_fmaf(dot, scale, bias) : dot * scale;
  else return has_bias ? dot + bias : dot;
}

constexpr int kBK = 64;          // K elements per staged step
constexpr int kGM = 8;           // m-tiles grouped per n-tile in the tile order

__device__ __forceinline__ void tile_of_block(int b, int m_tiles, int n_tiles, int& mt, int& nt) {
  const int total = m_tiles * n_tiles;
  const int full = total / 8 * 8;
  const int tile = b < full ? (b % 8) * (full / 8) + b / 8 : b;
  const int gm_max = m_tiles < kGM ? m_tiles : kGM;
  const int group = gm_max * n_tiles;
  const int g = tile / group;
  const int first_m = g * gm_max;
  const int gm = min(m_tiles - first_m, gm_max);
  const int in = tile - g * group;
  mt = first_m + in % gm;
  nt = in / gm;
}

// Lane exchanges of the butterfly below, all VALU except the 4-lane step:
// v_permlane16_swap exchanges the upper 16 lanes of each 32-lane half of one
// register with the lower 16 of another, so the larger of its two results is,
// in lanes l & 16 == 0, max(x[l], x[l ^ 16]) and otherwise max(y[l], y[l ^ 16]);
// DPP row_ror:8 and quad permutations read lane l ^ 8, l ^ 2 and l ^ 1.
template <int O>
__device__ __forceinline__ uint32_t lane_xor_u32(uint32_t v) {
  if constexpr (O == 8) return dpp_u32<0x128>(v);       // row_ror:8
  else if constexpr (O == 2) return dpp_u32<0x4E>(v);   // quad_perm 2,3,0,1
  else if constexpr (O == 1) return dpp_u32<0xB1>(v);   // quad_perm 1,0,3,2
  else return (uint32_t)__shfl_xor((int)v, O, 64);
}
template <class T>
__device__ __forceinline__ T vmax(T a, T b) { return a > b ? a : b; }

// v of lane l ^ 32: a permlane32 swap trades lanes [32, 64) of its first
// operand with lanes [0, 32) of its second, so with v in both a low lane
// finds its partner's value in the second result, a high lane in the first
__device__ __forceinline__ unsigned long long xor_lane_u64_32(unsigned long long v) {
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  const auto sl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto sh = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  const bool low = (threadIdx.x & 32) == 0;
  return ((unsigned long long)(low ? sh[1] : sh[0]) << 32) | (low ? sl[1] : sl[0]);
}

// Values are float or 64-bit keys, moved as 32-bit words.
template <class T, int O>
__device__ __forceinline__ T xor_lane(T v) {
  if constexpr (sizeof(T) == 8) {
    const uint32_t lo = lane_xor_u32<O>((uint32_t)v), hi = lane_xor_u32<O>((uint32_t)(v >> 32));
    return ((T)hi << 32) | lo;
  } else {
    return __uint_as_float(lane_xor_u32<O>(__float_as_uint(v)));
  }
}
template <class T>
__device__ __forceinline__ void swap16(T& x, T& y) {
  if constexpr (sizeof(T) == 8) {
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    x = ((T)hi[0] << 32) | lo[0];
    y = ((T)hi[1] << 32) | lo[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
  }
}

template <int O, int CNT, int P, class T>
__device__ __forceinline__ void half_wave_max_step(T (&v)[P], int lane) {
  if constexpr (O >= 1) {
    constexpr int H = CNT / 2;
    const bool upper = (lane & O) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      if constexpr (O == 16) {
        T x = v[i], y = v[i + H];
        swap16(x, y);
        v[i] = vmax(x, y);
      } else {
        const T t0 = vmax(v[i], xor_lane<T, O>(v[i]));
        const T t1 = vmax(v[i + H], xor_lane<T, O>(v[i + H]));
        v[i] = upper ? t1 : t0;
      }
    }
    half_wave_max_step<O / 2, H, P>(v, lane);
  }
}

// Transposing butterfly inside each 32-lane half of a wave: on entry lane l
// holds P values; after log2(32) exchanges lane (l & 31) holds the max over
// the half's 32 lanes of values (l & 31) * P/32 .. + P/32 - 1.
template <int P, class T>
__device__ __forceinline__ void half_wave_max_transpose(T (&v)[P], int lane) {
  static_assert(P >= 32 && P % 32 == 0, "values per lane");
  half_wave_max_step<16, P, P>(v, lane);
}

// A pointer that is the same in every lane, made visibly uniform (scalar
// registers) so that memory instructions can take it as their scalar base.
__device__ __forceinline__ const uint8_t* scalar_ptr(const void* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const uint8_t*>(((uint64_t)hi << 32) | lo);
}

typedef __attribute__((address_space(3))) void lds_void_t;

__device__ __forceinline__ int swz8(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// Copy addressing of the direct-to-LDS kernels.  With O32 every lane keeps
// its row's byte offset (below 4 GiB) in a 32-bit register and the step's
// base stays scalar: each copy is then the scalar-base + 32-bit-offset form
// of global_load_lds with no address arithmetic of its own (the empty asm
// keeps the compiler from folding the base into 64-bit lane addresses, which
// costs a 64-bit add per copy and chains the copies through one register
// pair).  Measured on dense_sub's cloud projection: 1106 -> 1033 us.

template <bool O32>
struct LaneAddr;
template <>
struct LaneAddr<true> {
  uint32_t off;
  __device__ __forceinline__ void set(const uint8_t*, int64_t o) { off = (uint32_t)o; }
  // base: the step's scalar base (from scalar_ptr)
  __device__ __forceinline__ void copy(const uint8_t* base, int64_t, lds_void_t* dst) {
    asm volatile("" : "+v"(off));
    __builtin_amdgcn_global_load_lds(base + off, dst, 16, 0, 0);
  }
  // the same, from `back` bytes before the lane's place
  __device__ __forceinline__ void copy_back(const uint8_t* base, int64_t, lds_void_t* dst, uint32_t back) {
    __builtin_amdgcn_global_load_lds(base + (off - back), dst, 16, 0, 0);
  }
};
template <>
struct LaneAddr<false> {
  const uint8_t* p;
  __device__ __forceinline__ void set(const uint8_t* base, int64_t o) { p = base + o; }
  __device__ __forceinline__ void copy(const uint8_t*, int64_t step, lds_void_t* dst) {
    __builtin_amdgcn_global_load_lds(p + step, dst, 16, 0, 0);
  }
  __device__ __forceinline__ void copy_back(const uint8_t*, int64_t step, lds_void_t* dst, uint32_t back) {
    __builtin_amdgcn_global_load_lds(p + step - back, dst, 16, 0, 0);
  }
};

// Clears the columns at and past `valid` (a multiple of 8 below kBK) of a
// staged tile of ROWS rows of kBK bf16, by NT threads.
template <int ROWS, int NT>
__device__ __forceinline__ void zero_tail(uint16_t* tile, int valid) {
  for (int i = threadIdx.x; i < ROWS * 8; i += NT) {
    const int row = i >> 3, c = i & 7;
    if (c * 8 >= valid)
      *reinterpret_cast<u32x4_t*>(tile + row * kBK + ((c ^ swz8(row)) << 3)) = u32x4_t{0u, 0u, 0u, 0u};
  }
}

// 32-bit copy offsets (LaneAddr<true>) when every row the copies address
// lies below 4 GiB of its operand's base.
inline bool copy_offsets_fit(const MfmaArgs& a) {
  constexpr int64_t kLim = 0xFFFFFFFFll;
  return a.w_rows > 0 && (int64_t)a.M * a.ldh * 2 <= kLim && a.w_rows * a.ldw_bytes <= kLim;
}

}  // namespace sph
