// AES-GCM seal and open of payload rows (eq. 19: the quantised payload is
// encrypted with AES-GCM under a key K and a nonce IV, with session, block
// and cache metadata as associated data).  AES per FIPS-197, GCM per NIST
// SP 800-38D with 96-bit IVs; every row is its own message.
//
// Key set-up (host, once per key): the S-box from its definition (inverse
// in GF(2^8) by discrete logarithms to the generator 3, then the affine map
// bit by bit), one 256-entry table T0[x] = (2S(x), S(x), S(x), 3S(x)) whose
// byte rotations give the other three column tables, the round keys, the
// hash key H = E_K(0^128) and the powers H^1 .. H^kGcmMaxPow.
//
// GHASH of a message with a AAD blocks, n ciphertext blocks and the length
// block is S = sum_k X_k H^(m-k+1), m = a + n + 1, so with the powers in a
// table every block's term is independent: ciphertext block j (0-based)
// contributes C_j H^(n+1-j).  k_gcm_blocks runs one thread per 16-byte block
// (counter-mode keystream from inc32 counters 2, 3, ... and the block's GHASH
// term) and xor-reduces the terms of its blocks, for small batches;
// k_gcm_bulk has each lane chain a few blocks of a larger batch; k_gcm_finish
// adds a row's partial sums and forms (seal) or checks (open) the tag
// E_K(J0) xor S.  Xor is exact and associative, so the result does not depend
// on the reduction order.  What bounds it is vector operations and LDS
// lookups, not memory: 320 rows of 60 KB move 38 MB (6 us).
#include <algorithm>
#include <cstring>
#include <type_traits>
#include <vector>

#include "sph_internal.h"

namespace sph {

namespace {

// ---------------------------------------------------------------------------
// host: S-box, tables, key schedule, powers of H
// ---------------------------------------------------------------------------

uint8_t xtime(uint8_t b) { return (uint8_t)((b << 1) ^ ((b & 0x80) ? 0x1B : 0x00)); }

void build_sbox(uint8_t sbox[256]) {
  // 3 generates the multiplicative group of GF(2^8): log / antilog tables
  uint8_t alog[255];
  int lg[256] = {0};
  uint8_t x = 1;
  for (int i = 0; i < 255; ++i) {
    alog[i] = x;
    lg[x] = i;
    x = (uint8_t)(x ^ xtime(x));  // x * 3
  }
  for (int a = 0; a < 256; ++a) {
    const uint8_t inv = a == 0 ? 0 : alog[(255 - lg[a]) % 255];
    // affine map: bit i of the result = b_i ^ b_(i+4) ^ b_(i+5) ^ b_(i+6) ^ b_(i+7) ^ c_i (indices mod 8)
    uint8_t r = 0;
    for (int i = 0; i < 8; ++i) {
      const int bit = ((inv >> i) ^ (inv >> ((i + 4) & 7)) ^ (inv >> ((i + 5) & 7)) ^
                       (inv >> ((i + 6) & 7)) ^ (inv >> ((i + 7) & 7)) ^ (0x63 >> i)) & 1;
      r = (uint8_t)(r | (bit << i));
    }
    sbox[a] = r;
  }
}

uint32_t rotr32(uint32_t v, int k) { return (v >> k) | (v << (32 - k)); }

}  // namespace

// words are big-endian: byte 0 of a column (row 0) is the most significant
__host__ __device__ __forceinline__ uint32_t gcm_rotr(uint32_t v, int k) {
  return (v >> k) | (v << (32 - k));
}

// One AES block: in/out as four big-endian column words.  te: the T0 table,
// sb: the S-box, rk: 4 (nr + 1) round-key words.
template <class TE, class SB, class RK>
__host__ __device__ __forceinline__ void aes_block(TE te, SB sb, RK rk, int nr, const uint32_t in[4],
                                                   uint32_t out[4]) {
  uint32_t s0 = in[0] ^ rk[0], s1 = in[1] ^ rk[1], s2 = in[2] ^ rk[2], s3 = in[3] ^ rk[3];
#pragma unroll
  for (int r = 1; r < nr; ++r) {
    // column c of the next state: T0[row 0 of column c] ^ T1[row 1 of c+1]
    // ^ T2[row 2 of c+2] ^ T3[row 3 of c+3] ^ round key (ShiftRows folded in)
    const uint32_t t0 = te[s0 >> 24] ^ gcm_rotr(te[(s1 >> 16) & 255], 8) ^
                        gcm_rotr(te[(s2 >> 8) & 255], 16) ^ gcm_rotr(te[s3 & 255], 24) ^ rk[4 * r];
    const uint32_t t1 = te[s1 >> 24] ^ gcm_rotr(te[(s2 >> 16) & 255], 8) ^
                        gcm_rotr(te[(s3 >> 8) & 255], 16) ^ gcm_rotr(te[s0 & 255], 24) ^ rk[4 * r + 1];
    const uint32_t t2 = te[s2 >> 24] ^ gcm_rotr(te[(s3 >> 16) & 255], 8) ^
                        gcm_rotr(te[(s0 >> 8) & 255], 16) ^ gcm_rotr(te[s1 & 255], 24) ^ rk[4 * r + 2];
    const uint32_t t3 = te[s3 >> 24] ^ gcm_rotr(te[(s0 >> 16) & 255], 8) ^
                        gcm_rotr(te[(s1 >> 8) & 255], 16) ^ gcm_rotr(te[s2 & 255], 24) ^ rk[4 * r + 3];
    s0 = t0; s1 = t1; s2 = t2; s3 = t3;
  }
  // last round: SubBytes and ShiftRows only
  auto last = [&](uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t k) {
    return (((uint32_t)sb[a >> 24]) << 24 | ((uint32_t)sb[(b >> 16) & 255]) << 16 |
            ((uint32_t)sb[(c >> 8) & 255]) << 8 | (uint32_t)sb[d & 255]) ^ k;
  };
  out[0] = last(s0, s1, s2, s3, rk[4 * nr]);
  out[1] = last(s1, s2, s3, s0, rk[4 * nr + 1]);
  out[2] = last(s2, s3, s0, s1, rk[4 * nr + 2]);
  out[3] = last(s3, s0, s1, s2, rk[4 * nr + 3]);
}

// Nibble tables of the product by y: the product is linear in its first
// factor, so x . y is the xor of the entries of x's nibbles.  The products of
// the single bits are y and its shifts.
static void nibble_tables(const uint32_t y[4], uint32_t* tab) {
  uint32_t bit[128][4];
  uint32_t v[4] = {y[0], y[1], y[2], y[3]};
  for (int i = 0; i < 128; ++i) {
    std::memcpy(bit[i], v, 16);
    const uint32_t lsb = 0u - (v[3] & 1u);
    v[3] = (v[3] >> 1) | (v[2] << 31);
    v[2] = (v[2] >> 1) | (v[1] << 31);
    v[1] = (v[1] >> 1) | (v[0] << 31);
    v[0] = (v[0] >> 1) ^ (0xE1000000u & lsb);
  }
  for (int p = 0; p < 32; ++p)
    for (int n = 0; n < 16; ++n)
      for (int w = 0; w < 4; ++w) {
        uint32_t r = 0;
        for (int b = 0; b < 4; ++b)
          if (n >> (3 - b) & 1) r ^= bit[4 * p + b][w];
        tab[4 * (16 * p + n) + w] = r;
      }
}

static void table_mul(const uint32_t x[4], const uint32_t* tab, uint32_t z[4]) {
  uint32_t r[4] = {0, 0, 0, 0};
  for (int p = 0; p < 32; ++p) {
    const uint32_t* e = tab + 4 * (16 * p + ((x[p >> 3] >> (28 - 4 * (p & 7))) & 15u));
    for (int w = 0; w < 4; ++w) r[w] ^= e[w];
  }
  std::memcpy(z, r, 16);
}

bool gcm_key_setup(const uint8_t* key, int key_bytes, std::vector<uint8_t>& dev_image, int& nr) {
  if (key_bytes != 16 && key_bytes != 32) return false;
  uint8_t sbox[256];
  build_sbox(sbox);
  uint32_t te[256];
  for (int x = 0; x < 256; ++x) {
    const uint8_t s = sbox[x], s2 = xtime(s), s3 = (uint8_t)(s2 ^ s);
    te[x] = ((uint32_t)s2 << 24) | ((uint32_t)s << 16) | ((uint32_t)s << 8) | s3;
  }
  const int nk = key_bytes / 4;
  nr = nk + 6;
  uint32_t w[60];
  for (int i = 0; i < nk; ++i)
    w[i] = ((uint32_t)key[4 * i] << 24) | ((uint32_t)key[4 * i + 1] << 16) |
           ((uint32_t)key[4 * i + 2] << 8) | key[4 * i + 3];
  uint8_t rc = 1;
  auto subword = [&](uint32_t v) {
    return ((uint32_t)sbox[v >> 24] << 24) | ((uint32_t)sbox[(v >> 16) & 255] << 16) |
           ((uint32_t)sbox[(v >> 8) & 255] << 8) | sbox[v & 255];
  };
  for (int i = nk; i < 4 * (nr + 1); ++i) {
    uint32_t t = w[i - 1];
    if (i % nk == 0) {
      t = subword(rotr32(t, 24)) ^ ((uint32_t)rc << 24);  // RotWord is a left byte rotation
      rc = xtime(rc);
    } else if (nk > 6 && i % nk == 4) {
      t = subword(t);
    }
    w[i] = w[i - nk] ^ t;
  }
  // device image: te | sbox | round keys | powers of H
  dev_image.assign(kGcmImageBytes, 0);
  std::memcpy(dev_image.data(), te, sizeof(te));
  std::memcpy(dev_image.data() + 1024, sbox, 256);
  std::memcpy(dev_image.data() + kGcmRkOffset, w, sizeof(uint32_t) * 4 * (nr + 1));
  const uint32_t zero[4] = {0, 0, 0, 0};
  uint32_t h[4];
  aes_block(te, sbox, w, nr, zero, h);
  uint32_t* pw = reinterpret_cast<uint32_t*>(dev_image.data() + kGcmPowOffset);  // pw[4e .. 4e+3] = H^e
  pw[0] = 0x80000000u;  // H^0 = 1
  std::memcpy(pw + 4, h, 16);
  std::vector<uint32_t> ht(32 * 16 * 4);
  nibble_tables(h, ht.data());
  for (int e = 2; e <= kGcmMaxPow; ++e) table_mul(pw + 4 * (e - 1), ht.data(), pw + 4 * e);
  nibble_tables(pw + 4 * 64, reinterpret_cast<uint32_t*>(dev_image.data() + kGcmTabOffset));
  return true;
}

// ---------------------------------------------------------------------------
// device
// ---------------------------------------------------------------------------

__device__ __forceinline__ void pack_be_words(const uint8_t b[16], uint32_t w[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k)
    w[k] = ((uint32_t)b[4 * k] << 24) | ((uint32_t)b[4 * k + 1] << 16) | ((uint32_t)b[4 * k + 2] << 8) |
           b[4 * k + 3];
}

// The first valid (1 ... 16) bytes at p, the rest zero.  Every load is made, at
// the last byte again past the end, so that the 16 are in flight together (a
// load in a branch of its own is waited for before the next).
__device__ __forceinline__ void load_be_words(const uint8_t* p, int valid, uint32_t w[4]) {
  uint8_t b[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) b[i] = p[min(i, valid - 1)];
#pragma unroll
  for (int i = 0; i < 16; ++i) b[i] = i < valid ? b[i] : 0;
  pack_be_words(b, w);
}

__device__ __forceinline__ void load_iv(const uint8_t* p, uint32_t w[3]) {
  uint32_t v[3];
  __builtin_memcpy(v, p, 12);
#pragma unroll
  for (int k = 0; k < 3; ++k) w[k] = __builtin_bswap32(v[k]);
}

// Segment of a message row that holds message byte p (p < L): the last
// segment starting at or before p, so empty segments are passed over.
__device__ __forceinline__ int seg_of(const GcmSegs& g, int64_t p, int64_t& start) {
  int s = 0;
  start = 0;
#pragma unroll
  for (int k = 0; k < kGcmMaxSegs - 1; ++k)
    if (k + 1 < g.nseg && p >= g.end[k]) {
      s = k + 1;
      start = g.end[k];
    }
  return s;
}

template <typename T>
__device__ __forceinline__ T* seg_ptr(T* const (&base)[kGcmMaxSegs], const int64_t (&ld)[kGcmMaxSegs],
                                      int s, int64_t row, int64_t off) {
  T* b = base[0];
  int64_t l = ld[0];
#pragma unroll
  for (int k = 1; k < kGcmMaxSegs; ++k)
    if (s == k) {
      b = base[k];
      l = ld[k];
    }
  return b + row * l + off;
}

// T0 sits in LDS with a copy for each of 32 lanes, and beside it T0 rotated by
// 16 bits: no two lanes of a half wave meet on a bank (one table would let any
// of them collide), a lookup's address is one byte permute (byte 1 the state's
// byte, byte 0 the lane's copy), and a column needs one rotation instead of
// three: 454 vector operations a block of AES-256.
struct GcmShared {
  uint32_t te[256 * 64];  // entry x of lane l at 64 x + l % 32, rotated at 32 more
};

__device__ __forceinline__ void stage_key(GcmShared& sh, const uint8_t* key_dev) {
  const uint32_t* te = reinterpret_cast<const uint32_t*>(key_dev);
  for (int i = threadIdx.x; i < 1024; i += blockDim.x) {
    uint32_t v = te[i >> 2];
    if (i & 2) v = gcm_rotr(v, 16);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<uint4*>(&sh.te[(i >> 2) * 64 + (i & 3) * 16 + 4 * q]) = make_uint4(v, v, v, v);
  }
}

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, (int)c, 0x96);
}

template <int NR>
__device__ __forceinline__ void aes_block_lds(const GcmShared& sh, const uint32_t* __restrict__ rk,
                                               const uint32_t (&in)[4], uint32_t (&out)[4]) {
  const uint32_t l4 = (threadIdx.x & 31u) * 4u;
  const uint8_t* te = reinterpret_cast<const uint8_t*>(sh.te);
  auto look = [&](uint32_t s, auto bytec, int rot) {
    constexpr uint32_t kSel = 0x0c0c0000u | ((4u + decltype(bytec)::value) << 8);
    return *reinterpret_cast<const uint32_t*>(te + __builtin_amdgcn_perm(s, l4, kSel) + 128 * rot);
  };
  using B0 = std::integral_constant<uint32_t, 0>;
  using B1 = std::integral_constant<uint32_t, 1>;
  using B2 = std::integral_constant<uint32_t, 2>;
  using B3 = std::integral_constant<uint32_t, 3>;
  uint32_t s[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) s[c] = in[c] ^ rk[c];
#pragma unroll
  for (int r = 1; r < NR; ++r) {
    uint32_t t[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t a = look(s[c], B3{}, 0), b = look(s[(c + 1) & 3], B2{}, 0);
      const uint32_t d = look(s[(c + 2) & 3], B1{}, 1), e = look(s[(c + 3) & 3], B0{}, 1);
      t[c] = gcm_rotr(b ^ e, 8) ^ xor3(a, d, rk[4 * r + c]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) s[c] = t[c];
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    // the S-box is bytes 1 and 2 of T0, 0 and 3 of the rotated entry
    const uint32_t a = look(s[c], B3{}, 1), b = look(s[(c + 1) & 3], B2{}, 0);
    const uint32_t d = look(s[(c + 2) & 3], B1{}, 0), e = look(s[(c + 3) & 3], B0{}, 1);
    const uint32_t ab = __builtin_amdgcn_perm(a, b, 0x07020c0cu), de = __builtin_amdgcn_perm(d, e, 0x0c0c0500u);
    out[c] = xor3(ab, de, rk[4 * NR + c]);
  }
}

// z = x . y in GF(2^128) by the comb method: the 255-bit product takes bit b of
// every word of x at a time, all words shifted once per b (28 operations for 4
// bits of x, 44 when each bit is reduced), then x^128 = 1 + x + x^2 + x^7.
__device__ __forceinline__ void gf128_mul_comb(const uint32_t x[4], const uint32_t y[4], uint32_t z[4]) {
  uint32_t p[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
  uint32_t xs[4] = {x[0], x[1], x[2], x[3]};  // bit 0 of each is the next
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
#pragma unroll
    for (int b = 0; b < 8; ++b) {
#pragma unroll
      for (int i = 7; i >= 1; --i) p[i] = __builtin_amdgcn_alignbit(p[i - 1], p[i], 1);
      p[0] >>= 1;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)xs[w], b, 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) p[w + i] ^= y[i] & m;
      }
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) xs[w] >>= 8;
  }
  // words 4 ... 7 times 1 + x + x^2 + x^7, and what that shifts out once more
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t h = p[4 + i], l = i > 0 ? p[3 + i] : 0u;
    z[i] = p[i] ^ h ^ __builtin_amdgcn_alignbit(l, h, 1) ^ __builtin_amdgcn_alignbit(l, h, 2) ^
           __builtin_amdgcn_alignbit(l, h, 7);
  }
  const uint32_t o = (p[7] << 31) ^ (p[7] << 30) ^ (p[7] << 25);
  z[0] ^= o ^ (o >> 1) ^ (o >> 2) ^ (o >> 7);
}

// xor over the wave's lanes, valid in lane 63
__device__ __forceinline__ uint32_t wave_xor_last(uint32_t v) {
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v ^= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// Y . G from the nibble tables in LDS: 32 independent lookups, no shifts.
__device__ __forceinline__ void mul_by_g(uint32_t y[4], const uint4* __restrict__ tab) {
  uint32_t r0 = 0u, r1 = 0u, r2 = 0u, r3 = 0u;
  const uint8_t* t = reinterpret_cast<const uint8_t*>(tab);
#pragma unroll
  for (int p = 0; p < 32; p += 2) {
    // a few entries at a time: one long xor would hold all 32 in registers
    if (p % 4 == 0) asm volatile("" : "+v"(r0), "+v"(r1), "+v"(r2), "+v"(r3));
    const uint32_t w = y[p >> 3];
    const int s0 = 24 - 4 * (p & 7), s1 = 20 - 4 * (p & 7);  // (nibble << 4) is the entry's byte offset
    const uint32_t o0 = w >> s0 & 0xF0u, o1 = (s1 >= 0 ? w >> (s1 & 31) : w << 4) & 0xF0u;
    const uint4 e = *reinterpret_cast<const uint4*>(t + 256 * p + o0);
    const uint4 f = *reinterpret_cast<const uint4*>(t + 256 * (p + 1) + o1);
    r0 = xor3(r0, e.x, f.x);
    r1 = xor3(r1, e.y, f.y);
    r2 = xor3(r2, e.z, f.z);
    r3 = xor3(r3, e.w, f.w);
  }
  y[0] = r0;
  y[1] = r1;
  y[2] = r2;
  y[3] = r3;
}

// One lane's data block of a row: its bytes are at in / out, from byte cut on
// (a block that straddles a segment boundary) at in2 / out2; a block over three
// or four segments (many) maps every byte on its own.
struct GcmBlock {
  int64_t p0;
  int valid, cut;
  bool many;
  const uint8_t *in, *in2;
  uint8_t *out, *out2;
};

__device__ __forceinline__ int64_t seg_end(const GcmSegs& segs, int s) {
  int64_t e = segs.end[0];
#pragma unroll
  for (int k = 1; k < kGcmMaxSegs; ++k)
    if (s == k) e = segs.end[k];
  return e;
}

__device__ __forceinline__ GcmBlock find_block(const GcmSegs& segs, int64_t L, int64_t row, int j) {
  GcmBlock b;
  b.p0 = (int64_t)j * 16;
  b.valid = (int)min<int64_t>(16, L - b.p0);
  int64_t st;
  const int s0 = seg_of(segs, b.p0, st);
  const int64_t e0 = seg_end(segs, s0);
  b.in = b.in2 = seg_ptr(segs.in, segs.ld_in, s0, row, b.p0 - st);
  b.out = b.out2 = seg_ptr(segs.out, segs.ld_out, s0, row, b.p0 - st);
  b.cut = 16;
  b.many = false;
  if (b.p0 + b.valid > e0) {
    const int s1 = seg_of(segs, e0, st);
    b.cut = (int)(e0 - b.p0);
    b.many = b.p0 + b.valid > seg_end(segs, s1);
    b.in2 = seg_ptr(segs.in, segs.ld_in, s1, row, b.p0 - st);
    b.out2 = seg_ptr(segs.out, segs.ld_out, s1, row, b.p0 - st);
  }
  return b;
}

// The bytes of a block that is not a whole one of one segment are all asked
// for before the first is used, the last one again past the message's end (a
// load in a branch of its own is waited for before the next).
__device__ __forceinline__ void load_block(const GcmSegs& segs, int64_t row, const GcmBlock& g, uint32_t x[4]) {
  if (g.cut == 16 && g.valid == 16) {  // one load at any alignment
    uint4 v;
    __builtin_memcpy(&v, g.in, 16);
    x[0] = __builtin_bswap32(v.x);
    x[1] = __builtin_bswap32(v.y);
    x[2] = __builtin_bswap32(v.z);
    x[3] = __builtin_bswap32(v.w);
  } else if (!g.many) {
    uint8_t b[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int k = min(i, g.valid - 1);
      b[i] = (k < g.cut ? g.in : g.in2)[k];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) b[i] = i < g.valid ? b[i] : 0;
    pack_be_words(b, x);
  } else {
    x[0] = x[1] = x[2] = x[3] = 0u;
#pragma unroll 1
    for (int i = 0; i < 16; ++i) {
      uint32_t v = 0u;
      if (i < g.valid) {
        int64_t st;
        const int s = seg_of(segs, g.p0 + i, st);
        v = *seg_ptr(segs.in, segs.ld_in, s, row, g.p0 + i - st);
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) x[k] = (x[k] << 8) | (x[k + 1] >> 24);
      x[3] = (x[3] << 8) | v;
    }
  }
}

__device__ __forceinline__ void store_block(const GcmSegs& segs, int64_t row, const GcmBlock& g,
                                            const uint32_t y[4]) {
  if (g.cut == 16 && g.valid == 16) {
    const uint4 v = make_uint4(__builtin_bswap32(y[0]), __builtin_bswap32(y[1]), __builtin_bswap32(y[2]),
                               __builtin_bswap32(y[3]));
    __builtin_memcpy(g.out, &v, 16);
  } else if (!g.many) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (i < g.valid) (i < g.cut ? g.out : g.out2)[i] = (uint8_t)(y[i >> 2] >> (24 - 8 * (i & 3)));
  } else {
    uint32_t v[4] = {y[0], y[1], y[2], y[3]};
#pragma unroll 1
    for (int i = 0; i < g.valid; ++i) {
      int64_t st;
      const int s = seg_of(segs, g.p0 + i, st);
      *seg_ptr(segs.out, segs.ld_out, s, row, g.p0 + i - st) = (uint8_t)(v[0] >> 24);
#pragma unroll
      for (int k = 0; k < 3; ++k) v[k] = (v[k] << 8) | (v[k + 1] >> 24);
      v[3] <<= 8;
    }
  }
}

// The GHASH input is the ciphertext: what was read when opening; when sealing
// what was written, zero past the message.
template <bool OPEN>
__device__ __forceinline__ void hash_input(const uint32_t x[4], const uint32_t y[4], int valid, uint32_t c[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) c[k] = OPEN ? x[k] : y[k];
  if (!OPEN && valid < 16) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (i >= valid) c[i >> 2] &= ~(0xFFu << (24 - 8 * (i & 3)));
  }
}

// Counter-mode output of data block j of a row, at g, and its GHASH input.  The
// bytes are asked for before the keystream is computed.
template <bool OPEN, int NR>
__device__ __forceinline__ void gcm_data_block(const GcmShared& sh, const uint32_t* __restrict__ rk,
                                               const GcmSegs& segs, const uint32_t ivw[3], int64_t row, int j,
                                               const GcmBlock& g, uint32_t c[4]) {
  uint32_t x[4], y[4], ks[4];
  load_block(segs, row, g, x);
  const uint32_t ctr[4] = {ivw[0], ivw[1], ivw[2], (uint32_t)(2 + j)};  // inc32 from J0 + 1
  aes_block_lds<NR>(sh, rk, ctr, ks);
#pragma unroll
  for (int k = 0; k < 4; ++k) y[k] = x[k] ^ ks[k];
  store_block(segs, row, g, y);
  hash_input<OPEN>(x, y, g.valid, c);
}

// AAD block u of a row (u < na, its power H^(m - u)), or the length block
// (u = na, its power H).
__device__ __forceinline__ void hash_other(const uint8_t* aad, int la, int64_t L, int u, uint32_t c[4]) {
  if (16 * u < la) {
    load_be_words(aad + (int64_t)u * 16, min(16, la - 16 * u), c);
  } else {
    const uint64_t abits = (uint64_t)la * 8, cbits = (uint64_t)L * 8;
    c[0] = (uint32_t)(abits >> 32);
    c[1] = (uint32_t)abits;
    c[2] = (uint32_t)(cbits >> 32);
    c[3] = (uint32_t)cbits;
  }
}

// A row's tag s: written (seal), or compared with the given one in constant
// time (open).
template <bool OPEN>
__device__ __forceinline__ void finish_row(const uint32_t s[4], uint8_t* tg, int32_t* ok) {
  if (OPEN) {
    uint32_t diff = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) diff |= (uint32_t)((uint8_t)(s[i >> 2] >> (24 - 8 * (i & 3))) ^ tg[i]);
    *ok = diff == 0 ? 1 : 0;
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) tg[i] = (uint8_t)(s[i >> 2] >> (24 - 8 * (i & 3)));
  }
}

// GHASH of a message of na AAD blocks and n data blocks is the sum of the
// m = na + n + 1 terms X_k . H^(m+1-k) (k = 1..m, X_m the length block), and
// the tag is that sum xor E_K(J0).  Every term is independent given the
// powers of H.  Workgroup q of a row (grid: parts x rows) covers the data
// blocks [q T, (q + 1) T), one to each of its T threads, and workgroup xpart
// the other na + 2 terms besides, in the threads after its last block: such a
// workgroup takes the same one pass (or a second one, if its blocks leave too
// few threads).  Each workgroup xor-reduces its terms into one 16-byte
// partial of the row, or into its tag where the row has one workgroup (which
// saves the launch of k_gcm_finish: 26 rows of 3433 B 13.2 -> 9.7 us).
// NR: 10 rounds (AES-128) or 14 (AES-256), fixed so that the rounds unroll
template <bool OPEN, int NR>
__global__ __launch_bounds__(1024) void k_gcm_blocks(const uint8_t* __restrict__ key_dev, const GcmSegs segs,
                                                     int64_t L, int n, int xpart, const uint8_t* __restrict__ iv,
                                                     const uint8_t* __restrict__ aad, int64_t ld_aad, int la,
                                                     uint32_t* __restrict__ partial, int nparts,
                                                     uint8_t* __restrict__ tag, int32_t* __restrict__ ok) {
  __shared__ __attribute__((aligned(16))) GcmShared sh;
  __shared__ uint32_t red[16][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = blockIdx.y;
  const uint32_t* rk = reinterpret_cast<const uint32_t*>(key_dev + kGcmRkOffset);
  const uint32_t* pw = reinterpret_cast<const uint32_t*>(key_dev + kGcmPowOffset);
  const int na = (la + 15) / 16, m = na + n + 1;
  const int j0 = blockIdx.x * blockDim.x, nd = max(0, min(n - j0, (int)blockDim.x));
  const int items = nd + ((int)blockIdx.x == xpart ? na + 2 : 0);
  uint32_t ivw[3], t[4] = {0u, 0u, 0u, 0u};
  load_iv(iv + row * 12, ivw);
  stage_key(sh, key_dev);
  __syncthreads();
  for (int it = tid; it < items; it += blockDim.x) {
    const int j = j0 + it, u = it - nd;  // data block j (u < 0) or other term u
    GcmBlock g;
    uint32_t x[4] = {0u, 0u, 0u, 0u}, y[4], c[4], r[4];
    int e = 0;  // E_K(J0): times 1
    if (u < 0) {
      g = find_block(segs, L, row, j);
      load_block(segs, row, g, x);
      e = n + 1 - j;
    } else if (u <= na) {
      hash_other(aad + row * ld_aad, la, L, u, x);
      e = u < na ? m - u : 1;
    }
    const uint32_t h4[4] = {pw[4 * e], pw[4 * e + 1], pw[4 * e + 2], pw[4 * e + 3]};
    const uint32_t ctr[4] = {ivw[0], ivw[1], ivw[2], u < 0 ? (uint32_t)(2 + j) : 1u};  // inc32 from J0 + 1; J0
    aes_block_lds<NR>(sh, rk, ctr, y);
#pragma unroll
    for (int k = 0; k < 4; ++k) y[k] ^= x[k];
    if (u < 0) {
      store_block(segs, row, g, y);
      hash_input<OPEN>(x, y, g.valid, c);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) c[k] = u <= na ? x[k] : y[k];
    }
    gf128_mul_comb(c, h4, r);
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] ^= r[k];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    t[k] = wave_xor_last(t[k]);
    if (lane == 63) red[wave][k] = t[k];
  }
  __syncthreads();
  if (nparts == 1) {
    if (tid == 0) {
      uint32_t s[4] = {0u, 0u, 0u, 0u};
      for (int w = 0; w < (int)blockDim.x / 64; ++w)
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] ^= red[w][k];
      finish_row<OPEN>(s, tag + row * 16, ok + row);
    }
  } else if (tid < 4) {
    uint32_t v = 0u;
    for (int w = 0; w < (int)blockDim.x / 64; ++w) v ^= red[w][tid];
    partial[(row * nparts + blockIdx.x) * 4 + tid] = v;
  }
}

// Larger batches.  A wave takes pieces of 64 * chain data blocks of a row, lane
// by lane, and needs no other wave: lane l chains blocks l + 64 i by Horner's
// rule in H^64 and ends in one comb product by its power of H; the wave's sum
// meets the row's others by atomic xor in the row's partial (zeroed before).
// The piece's last 64 places are its last blocks (places before its first
// block are zeros), so every piece ends with the same powers.  Pieces go round
// the workgroups wave by wave, so the CUs' shares differ by one wave.
// After the pieces come the rows' other terms, one to a lane: E_K(J0) of
// all rows, then their length and AAD blocks.
//
// A block is 454 vector operations of AES-256, 152 of the product by H^64 and
// about 50 of input and output, and its 224 + 32 lookups keep the LDS half as
// long; the last product is 1100.  320 rows of 60 KB: 100 us as chains of 16 in
// 320 workgroups of 256 threads (5 waves to 4 SIMDs, all latency), 49 now; with
// a workgroup's 16 waves' sums folded by a tree of products between barriers
// instead of a last product in each wave, 83.
constexpr int kBulkThreads = 1024;
constexpr int kBulkWaves = kBulkThreads / 64;

template <bool OPEN, int NR>
__global__ __launch_bounds__(kBulkThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_gcm_bulk(
    const uint8_t* __restrict__ key_dev, const GcmSegs segs, int64_t L, int n, int rows, int chain, int per_row,
    const uint8_t* __restrict__ iv, const uint8_t* __restrict__ aad, int64_t ld_aad, int la,
    uint32_t* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) GcmShared sh;
  __shared__ uint4 tab[32 * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t* rk = reinterpret_cast<const uint32_t*>(key_dev + kGcmRkOffset);
  const uint32_t* pw = reinterpret_cast<const uint32_t*>(key_dev + kGcmPowOffset);
  if (tid < 512) tab[tid] = reinterpret_cast<const uint4*>(key_dev + kGcmTabOffset)[tid];
  stage_key(sh, key_dev);
  __syncthreads();
  const int na = (la + 15) / 16, pieces = rows * per_row;
  const int more = (rows + 63) / 64, others = more + (int)(((int64_t)rows * (na + 1) + 63) / 64);
  // (the second half of the workgroups, the CUs' second ones, begins with the
  // third SIMD)
  const int turn = (wave + (blockIdx.x >= gridDim.x / 2 ? 2 : 0)) % kBulkWaves;
  for (int p = blockIdx.x + gridDim.x * turn; p < pieces + others; p += gridDim.x * kBulkWaves) {
    if (p < pieces) {
      const int row = p / per_row, j0 = (p - row * per_row) * 64 * chain, j1 = min(n, j0 + 64 * chain);
      const int ch = (j1 - j0 + 63) / 64;
      uint32_t ivw[3], y[4] = {0u, 0u, 0u, 0u};
      load_iv(iv + (int64_t)row * 12, ivw);
      for (int i = 0; i < ch; ++i) {
        const int jw = j1 - 64 * (ch - i), j = jw + lane;
        if (i > 0) mul_by_g(y, tab);
        if (j >= j0) {
          uint32_t c[4];
          // 64 whole blocks of one segment: found once for the wave
          GcmBlock g = find_block(segs, L, row, max(jw, 0));
          const int64_t end = g.p0 + 1024;
          int64_t st;
          if (jw >= j0 && end <= L && end <= seg_end(segs, seg_of(segs, g.p0, st))) {
            g.in += lane * 16;
            g.out += lane * 16;
            g.cut = g.valid = 16;
          } else {
            g = find_block(segs, L, row, j);
          }
          gcm_data_block<OPEN, NR>(sh, rk, segs, ivw, row, j, g, c);
#pragma unroll
          for (int k = 0; k < 4; ++k) y[k] ^= c[k];
        }
      }
      const uint32_t* hp = pw + 4 * (n + 2 - j1 + 63 - lane);  // the last block's power is n + 1 - (j1 - 1)
      const uint32_t h4[4] = {hp[0], hp[1], hp[2], hp[3]};
      uint32_t t[4];
      gf128_mul_comb(y, h4, t);
      uint32_t sum = 0u;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)wave_xor_last(t[k]), 63);
        if (lane == k) sum = v;
      }
      if (lane < 4) atomicXor(&partial[(int64_t)row * 4 + lane], sum);
    } else {
      const int64_t w = p - pieces, i = w < more ? w * 64 + lane : (w - more) * 64 + lane;
      const int64_t row = w < more ? i : i / (na + 1);
      const int u = w < more ? na + 1 : (int)(i - row * (na + 1));
      uint32_t t[4] = {0u, 0u, 0u, 0u};
      if (row < rows) {
        uint32_t c[4];
        if (u > na) {
          uint32_t ivw[3];
          load_iv(iv + row * 12, ivw);
          const uint32_t j0b[4] = {ivw[0], ivw[1], ivw[2], 1u};
          aes_block_lds<NR>(sh, rk, j0b, t);
        } else {
          hash_other(aad + row * ld_aad, la, L, u, c);
          const uint32_t* hp = pw + 4 * (u < na ? na + n + 1 - u : 1);
          const uint32_t h4[4] = {hp[0], hp[1], hp[2], hp[3]};
          gf128_mul_comb(c, h4, t);
        }
      }
      // a row's terms are in lanes next to each other, the last of which adds
      // their sum (with an atomic for every term a row's met one by one: 667 rows
      // of 37 B with 1 KB of AAD 53 -> 19 us, 2212 of 27 KB 175 -> 116)
      bool last = true;
      if (w >= more && na > 0) {
#pragma unroll
        for (int o = 1; o < 64; o *= 2) {
          const int r = __shfl_up((int)row, o, 64);
          const bool mine = lane >= o && r == (int)row;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint32_t v = __shfl_up(t[k], o, 64);
            t[k] ^= mine ? v : 0u;
          }
        }
        const int next = __shfl_down((int)row, 1, 64);  // (by every lane)
        last = lane == 63 || next != (int)row;
      }
      if (last && row < rows)
#pragma unroll
        for (int k = 0; k < 4; ++k) atomicXor(&partial[row * 4 + k], t[k]);
    }
  }
}

__global__ __launch_bounds__(256) void k_gcm_zero(uint32_t* __restrict__ p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// One thread per row: the xor of the row's partials is its tag.
template <bool OPEN>
__global__ __launch_bounds__(256) void k_gcm_finish(int rows, const uint32_t* __restrict__ partial,
                                                    int nparts, uint8_t* __restrict__ tag,
                                                    int32_t* __restrict__ ok) {
  const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (row >= rows) return;
  uint32_t s[4] = {0u, 0u, 0u, 0u};
  for (int p = 0; p < nparts; ++p)
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] ^= partial[(row * nparts + p) * 4 + k];
  finish_row<OPEN>(s, tag + row * 16, ok + row);
}

// Waves of k_gcm_bulk that take the rows' other terms.
static int64_t bulk_others(int64_t rows, int64_t na) { return (rows + 63) / 64 + (rows * (na + 1) + 63) / 64; }

// Blocks a lane of k_gcm_bulk chains.  A wave's time is that of its chain and
// of its last product, which costs about 2 blocks; the waves of a SIMD share
// it once there are 5 of them, below that a chain's latency is the time.
// (us, 32-byte keys, chains of 1 / 2 / 3 / 4 / 5 / 7: 320 rows of 60 KB 77, 61,
// 52, 49, 49, 58; 1024 of 16 KB 70, 59, 49, 54, 51, 57; 155 of 45 KB 38, 34,
// 33, 34, 37, 45.)
int gcm_bulk_chain(int64_t rows, int64_t n, int64_t na) {
  const int64_t others = bulk_others(rows, na);
  int best = 1;
  double t_best = 0;
  for (int k = 1; k <= kGcmMaxChain; ++k) {
    const int64_t waves = rows * ((n + 64 * k - 1) / (64 * k)) + others;
    const double t = (double)std::max<int64_t>(5, (waves + 4 * kCUs - 1) / (4 * kCUs)) * (k + 2);
    if (k == 1 || t < t_best) {
      best = k;
      t_best = t;
    }
  }
  return best;
}

hipError_t launch_gcm(bool open, const uint8_t* key_dev, int nr, const GcmSegs& segs, int rows,
                      const uint8_t* iv, const uint8_t* aad, int64_t ld_aad, int la, uint8_t* tag,
                      int32_t* ok, uint32_t* partial, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (segs.nseg < 1 || segs.nseg > kGcmMaxSegs || rows > 65535 || la < 0 || la > kGcmMaxAad)
    return hipErrorInvalidValue;
  const int64_t L = segs.end[segs.nseg - 1];
  const int n = (int)((L + 15) / 16);
  const int chain = gcm_chain(rows, n);
  int xpart = 0;
  const int nparts = gcm_parts(n, (la + 15) / 16, chain, &xpart);
  if (nr != 10 && nr != 14) return hipErrorInvalidValue;
  int sums = nparts;  // partials per row
  // One pass of one block a thread while the workgroups of up to 1024 threads
  // that the partials allow are all on the chip at once (two a CU): 13 us for
  // 26 rows of 3.4 KB, 14 for 16 of 49 KB, 21 for 64 of 32 KB, where k_gcm_bulk
  // takes 18, 22 and 21; and 34 for 5000 of 160 B, where k_gcm_blocks would
  // take 86.
  if (chain <= 4 && (int64_t)rows * nparts <= 2 * kCUs) {
    auto kern = open ? (nr == 10 ? k_gcm_blocks<true, 10> : k_gcm_blocks<true, 14>)
                     : (nr == 10 ? k_gcm_blocks<false, 10> : k_gcm_blocks<false, 14>);
    // one workgroup for a row of up to 512 terms too, which saves the second
    // launch: 16 rows of 8000 B 12.5 -> 11.1 us, 120 of 4200 B 14.0 -> 12.6; 1024
    // threads take longer than that (3 rows of 13 KB 12.4 -> 17.0)
    const int all = n + (la + 15) / 16 + 2;
    const bool one = nparts == 1 || all <= 512;
    const int threads = one ? std::min(1024, std::max(kGcmStride, (all + 63) / 64 * 64)) : kGcmStride * chain;
    launch_kernel(kern, dim3(one ? 1 : nparts, rows), dim3(threads), 0, s, key_dev, segs, L, n, one ? 0 : xpart, iv,
                  aad, ld_aad, la, partial, one ? 1 : nparts, tag, ok);
    if (one) return hipGetLastError();
  } else {
    const int64_t na = (la + 15) / 16, others = bulk_others(rows, na);
    const int c = gcm_bulk_chain(rows, n, na), per_row = (n + 64 * c - 1) / (64 * c);
    auto kern = open ? (nr == 10 ? k_gcm_bulk<true, 10> : k_gcm_bulk<true, 14>)
                     : (nr == 10 ? k_gcm_bulk<false, 10> : k_gcm_bulk<false, 14>);
    launch_kernel(k_gcm_zero, dim3((rows * 4 + 255) / 256), dim3(256), 0, s, partial, rows * 4);
    launch_kernel(kern, dim3((unsigned)std::min<int64_t>(rows * (int64_t)per_row + others, 2 * kCUs)),
                  dim3(kBulkThreads), 0, s, key_dev, segs, L, n, rows, c, per_row, iv, aad, ld_aad, la, partial);
    sums = 1;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int fb = (rows + 255) / 256;
  if (open)
    launch_kernel(k_gcm_finish<true>, dim3(fb), dim3(256), 0, s, rows, partial, sums, tag, ok);
  else
    launch_kernel(k_gcm_finish<false>, dim3(fb), dim3(256), 0, s, rows, partial, sums, tag, ok);
  return hipGetLastError();
}

}  // namespace sph
