// Products by the challenge on the matrix cores.
//
// The challenge c has tau coefficients of +-1 and the polynomials it multiplies
// (s1, s2, t0, t1) are small, so c p mod (X^256 + 1) fits 32-bit integers
// exactly and needs no transform: coefficient i is sum_j T[i][j] p[j] with the
// negacyclic Toeplitz matrix T[i][j] = c[i - j] (i >= j), -c[256 + i - j]
// (i < j).  One wavefront multiplies T by 16 int8 rows at a time with
// v_mfma_i32_16x16x64_i8 (D = rows x T^t, 64 instructions per 16 rows).
//
// Rows: a tile holds 16 int8 rows of 256; lane l's accumulator acc[I][r] is
// coefficient 16 I + (l & 15) of row 4 (l >> 4) + r.  With rows 4 g + r = part
// r of polynomial g, the 16-lane group g therefore receives all the parts of
// its own polynomial in the strided layout of ntt.h (register I = coefficient
// t + 16 I), next to y, w and the INTT's output.
//
// T in LDS: every fragment is a 16-byte window of f[m] = c[255 - m] (m < 256),
// -c[511 - m] (m >= 256): lane (i, kg) of the block (I, J) needs f from
// 15 - i + 16 u on, u = 4 J + kg - I + 15.  Copy b of f starts at byte b, so
// that every window is word-aligned in copy (15 - i) & 3; copies are 136 words
// apart, which puts the words that 32 lanes read at once into 32 different
// banks.  Only w = 4 J - I matters for the address: 28 windows feed the 64
// products (20 + 20 when they are made in two halves, which holds 32
// accumulator registers instead of 64).  (16 copies, one per i, make every
// window one aligned 16-byte read but take 8.4 KB of LDS per wavefront instead
// of 2.3 and three times the instructions to build.)
#pragma once
#include "common.h"
#include "poly.h"

namespace dil {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int TOEP_ROW = 136;             // words of one shifted copy: 127 used, padded
constexpr int TOEP_WORDS = 4 * TOEP_ROW;  // one wavefront's copies

// Build the four shifted copies from the dense challenge (cw: the lane's four
// coefficients 4 lane .. 4 lane + 3) with one wavefront.  f: 129 words of LDS scratch.
__device__ __forceinline__ void toep_build(uint32_t cw, uint32_t *ct, uint32_t *f, int lane) {
  const uint32_t rev = __builtin_amdgcn_perm(cw, cw, 0x00010203u);  // bytes reversed
  f[63 - lane] = rev;
  // bytes of {-1, 0, 1} negated: flip the upper seven bits of the non-zero ones
  f[127 - lane] = rev ^ ((rev & 0x01010101u) * 0xFEu);
  if (lane == 0) f[128] = 0;  // read, never used
  wave_sync();
  const int b = lane & 3, q = lane >> 2;  // copy b, words 8 q .. 8 q + 7
  uint32_t x[9];
#pragma unroll
  for (int k = 0; k < 9; k++) x[k] = f[8 * q + k];
  v4i *dst = (v4i *)(ct + b * TOEP_ROW + 8 * q);
#pragma unroll
  for (int u = 0; u < 2; u++) {
    v4i o;
#pragma unroll
    for (int k = 0; k < 4; k++) o[k] = (int)__builtin_amdgcn_alignbyte(x[4 * u + k + 1], x[4 * u + k], b);
    dst[u] = o;
  }
  wave_sync();
}

// the lane's part of a tile's 16 rows (rows 256 bytes apart, 16-byte aligned)
__device__ __forceinline__ void toep_load(v4i s[4], const int8_t *tile, int lane) {
  const int8_t *p = tile + (lane & 15) * N + 16 * (lane >> 4);
#pragma unroll
  for (int J = 0; J < 4; J++) s[J] = *(const v4i *)(p + 64 * J);
}

// Accumulators I = I0 .. I0 + NI - 1 of a tile.
template <int I0, int NI>
__device__ __forceinline__ void toep_mul(v4i acc[NI], const v4i s[4], const uint32_t *ct, int lane) {
  const int o = 15 - (lane & 15);
  const uint32_t *row = ct + (o & 3) * TOEP_ROW + (o >> 2) + 4 * (lane >> 4);
#pragma unroll
  for (int I = 0; I < NI; I++) acc[I] = v4i{0, 0, 0, 0};
#pragma unroll
  for (int w = -(I0 + NI - 1); w <= 12 - I0; w++) {
    const uint32_t *p = row + 4 * (w + 15);
    const v4i b = {(int)p[0], (int)p[1], (int)p[2], (int)p[3]};
#pragma unroll
    for (int J = 0; J < 4; J++) {
      const int I = 4 * J - w - I0;
      if (I >= 0 && I < NI) acc[I] = __builtin_amdgcn_mfma_i32_16x16x64_i8(s[J], b, acc[I], 0, 0, 0);
    }
  }
}

// Tiles of the Sign secrets: part 0 = s1, 1 = s2, 2 / 3 = t0 = lo + 64 hi (lo
// in [-32, 31], hi in [-64, 64]) of the tile's polynomials 4 T + g; absent
// rows are zero.
template <int LV>
constexpr int sec_tiles() { return ((Lv<LV>::K > Lv<LV>::L ? Lv<LV>::K : Lv<LV>::L) + 3) / 4; }
constexpr int TILE_BYTES = 16 * N;
template <int LV>
constexpr size_t sec_bytes() { return (size_t)sec_tiles<LV>() * TILE_BYTES; }

// Verify's t1 = lo + 32 hi (5 bits each), one tile for all K <= 8 polynomials:
// parts 0 / 1 of group g are lo / hi of polynomial g, parts 2 / 3 those of
// polynomial g + 4.  The lane's operands come straight from the packed public
// key: 16 coefficients are five of its words.  t1 = pk + 32 bytes.
template <int LV>
__device__ __forceinline__ void toep_load_t1(v4i s[4], const uint32_t *t1, int lane) {
  constexpr int K = Lv<LV>::K, T1W = 320 / 4;
  const int n = lane & 15, kg = lane >> 4, p = (n >> 2) + 4 * ((n >> 1) & 1), sh = 5 * (n & 1);
  const uint32_t *src = t1 + (p < K ? p : 0) * T1W + 5 * kg;
#pragma unroll
  for (int J = 0; J < 4; J++) {
    uint32_t w[5];
#pragma unroll
    for (int q = 0; q < 5; q++) w[q] = src[20 * J + q];
#pragma unroll
    for (int d = 0; d < 4; d++) {
      // four fields of 10 bits from bit 40 d = 32 d + 8 d on: three in x, the last in y
      // 14 / 6 / 14 / 22 bits up; each gives the five bits that start at its bit sh
      const uint32_t x = __builtin_amdgcn_alignbit(w[d + 1], w[d], 8 * d + sh);
      const uint32_t y = (d == 0 ? __builtin_amdgcn_alignbit(w[1], w[0], 16) : w[d + 1]) >> sh;
      const int up = d == 1 ? 6 : d == 3 ? 22 : 14;
      const uint32_t v = (x & 0x1Fu) | ((x >> 2) & 0x1F00u) | ((x >> 4) & 0x1F0000u) | ((y << (24 - up)) & 0x1F000000u);
      s[J][d] = p < K ? (int)v : 0;
    }
  }
}
// x - 2^13 c t1 mod q in [0, q) of one coefficient (|x| < q): |c t1| <= tau 1023 <
// 2^16, so the difference fits 31 bits, and z - (z + 2^22 >> 23) q lies in (-q, q)
// for |z| < 2^31 - 2^22 (2^23 = q + 2^13 - 1).
__device__ __forceinline__ int32_t sub_ct1(int32_t x, int32_t ct1) {
  int32_t z = x - __mul24(ct1, 1 << D);
  z -= __mul24((z + (1 << 22)) >> 23, Q);
  return canon(z);
}

}  // namespace dil
