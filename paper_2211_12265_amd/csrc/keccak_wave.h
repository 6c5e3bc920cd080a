// Keccak-f[1600] with one state on a whole wavefront, for the smallest batches:
// as the 16-lane form (keccak_row.h), but row y of the wavefront holds plane y
// in one register and every row holds plane 4 in a second one, so that a round
// is 24 VALU and 7 LDS instructions instead of 34 and 14.
//   theta  column parity by two lane swaps across the rows; the rest as on a row;
//   rho, pi  through LDS; plane 4 is written by row 0 only and read by all rows;
//   chi    as on a row.
// A permutation of a lone wavefront takes 2.5 us against 3.1 us on a row, 1,024
// states 2.8 against 3.2 us and 2,048, two wavefronts per SIMD, 3.4 us on both;
// 4,096 take 5.1 us against 4.4 us: rows take over above 2,048 (WAVE_STATES).
// The mu chains of 613 messages of up to 6 KB take 124 us (rows 213, pairs 493).
// Lone wavefronts wait for each instruction's result, the four rounds of one loop
// step save a branch each (2.65 us without), and the round constants come from
// LDS, where lanes that take none read zeros (scalar loads: 2.65 us).
#pragma once
#include "keccak_pair.h"

namespace dil {

template <int CTRL>
__device__ __forceinline__ uint32_t row_dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
// rotation amounts of the words that land in plane y, sheets 0 .. 4, six bits each
constexpr uint32_t row_rot(int y) {
  uint32_t v = 0;
  for (int x = 0; x < 5; x++) v |= (uint32_t)kc_rho((3 * y + x) % 5 + 5 * x) << (6 * x);
  return v;
}
// column parities of neighbouring sheets, given the lane's own: theta's d
__device__ __forceinline__ uint32_t row_theta(uint32_t c, uint32_t &cm) {
  cm = row_dpp<0x112>(c);  // lane l - 2
  // lane l + 2; lanes 8 .. 11 from lane l - 8
  const uint32_t cp = (uint32_t)__builtin_amdgcn_update_dpp((int)row_dpp<0x102>(c), (int)c, 0x118, 0xF, 0x4, false);
  return __builtin_amdgcn_alignbit(cp, pair_swap(cp), 31);
}

constexpr int KECCAK_LDS = 352;  // words of LDS per wavefront of either form
constexpr int KECCAK_RC = 256;   // of which the round constants, and as many zeros
// Writes them with the LANES lanes of one state (the wavefront's other states may
// not be there); where a lane that takes the constants' half h, or none, reads its own.
template <int LANES>
__device__ __forceinline__ const uint32_t *kc_rc_lds(uint32_t *lds, int l, bool takes, int h) {
#pragma unroll
  for (int i = 0; i < 48; i += LANES)
    if (i + l < 48) {
      const int w = i + l;
      lds[KECCAK_RC + w] = w & 1 ? kKRC.hi[w >> 1] : kKRC.lo[w >> 1];
      lds[KECCAK_RC + 48 + w] = 0;
    }
  wave_sync();
  return lds + KECCAK_RC + (takes ? h : 48);
}
constexpr uint32_t WAVE_STATES = 2048;

// the lane's constants; L: the wavefront's KECCAK_LDS words (50 of the state, a
// dump for unkept words, the round constants)
struct WaveKeccak {
  static constexpr int NR = 2, NA = 1, ND = 1;  // registers; those with words of the rate; with words 0 .. 9
  static constexpr int LANES = 64, STATES = 1;
  uint32_t *L;
  int x, h, row, l;
  int st = 0;
  bool own;                // holds words of its own (lanes 10 .. 15 of a row are copies)
  int w0, w1;              // where the lane keeps its words
  int p0, q0, p1, q1;      // high and low operand of the rotations that yield its words
  uint32_t s0, s1;         // their amounts
  const uint32_t *rc;
  __device__ __forceinline__ WaveKeccak(uint32_t *lds, int lane) {
    constexpr int DUMP = 50;
    L = lds;
    l = lane & 63;
    row = l >> 4;
    const int c = l & 15, m = c < 10 ? c : c - 10;
    x = m >> 1;
    h = m & 1;
    own = c < 10;
    const bool keep = c >= 2 && c < 12;
    w0 = keep ? 2 * (x + 5 * row) + h : DUMP + l;
    w1 = keep && row == 0 ? 2 * (x + 20) + h : DUMP + l;
    constexpr uint32_t rot[5] = {row_rot(0), row_rot(1), row_rot(2), row_rot(3), row_rot(4)};
    place(row, row < 2 ? (row == 0 ? rot[0] : rot[1]) : (row == 2 ? rot[2] : rot[3]), p0, q0, s0);
    place(4, rot[4], p1, q1, s1);
    rc = kc_rc_lds<LANES>(L, l, x == 0 && row == 0, h);
  }
  // where plane Y is read from: word (sx, x) with sx = x + 3 Y mod 5
  __device__ __forceinline__ void place(int Y, uint32_t rot, int &p, int &q, uint32_t &s) {
    int sx = x + (Y == 0 ? 0 : Y == 1 ? 3 : Y == 2 ? 1 : Y == 3 ? 4 : 2);
    sx = sx >= 5 ? sx - 5 : sx;
    const int n = (int)((rot >> (6 * x)) & 63u);
    const int mine = 2 * (sx + 5 * x) + h, other = mine + 1 - 2 * h;
    p = n > 32 ? other : mine;
    q = n == 0 || n > 32 ? mine : other;
    s = (uint32_t)-n & 31u;  // 32 - n, 64 - n, or 0
  }
  // 8-byte word index of register y, and the 32-bit word of it that this lane holds
  __device__ __forceinline__ int word(int y) const { return y == 0 ? 5 * row + x : 20 + x; }
  __device__ __forceinline__ int half_word(int y) const { return 2 * word(y) + h; }
  // whether `v` holds on a lane of the state
  __device__ __forceinline__ bool any(bool v) const { return __ballot(v) != 0; }
};

__device__ __forceinline__ void keccak_f_coop(uint32_t a[2], const WaveKeccak &k) {
  const uint32_t *rc = k.rc;
#pragma unroll 4
  for (int ir = 0; ir < 24; ir++) {
    const uint32_t rcv = rc[0];
    rc += 2;
    const auto e = __builtin_amdgcn_permlane16_swap(a[0], a[0], false, false);
    const uint32_t f = e[0] ^ e[1];
    const auto g = __builtin_amdgcn_permlane32_swap(f, f, false, false);
    uint32_t cm;
    const uint32_t r = row_theta(xor3(g[0], g[1], a[1]), cm);
    k.L[k.w0] = xor3(a[0], cm, r);
    k.L[k.w1] = xor3(a[1], cm, r);
    wave_sync();
    const uint32_t b0 = __builtin_amdgcn_alignbit(k.L[k.p0], k.L[k.q0], k.s0);
    const uint32_t b1 = __builtin_amdgcn_alignbit(k.L[k.p1], k.L[k.q1], k.s1);
    wave_sync();
    a[0] = chi3(b0, row_dpp<0x102>(b0), row_dpp<0x104>(b0)) ^ rcv;
    a[1] = chi3(b1, row_dpp<0x102>(b1), row_dpp<0x104>(b1));
  }
}

// SampleInBall on a wavefront whose state holds the first SHAKE256 block of
// ctilde; c: 256 bytes of LDS, 4-byte aligned.  Lane k follows the sign that
// step k places: at b_k until a later step whose index is that place moves it
// to its own i; no step reads the array.  The bytes come from lanes, so a step
// is some 12 instructions without a wait for LDS (5 -> 2 us for 49 steps).
template <int TAU>
__device__ __forceinline__ void sample_in_ball_coop(uint32_t a[2], const WaveKeccak &k, int8_t *c, uint32_t *) {
  static_assert(TAU <= 64, "one step per lane");
  auto words = [&]() {  // lane j: word j of the block
    if (k.own && k.word(0) < RATE256 / 8) k.L[k.half_word(0)] = a[0];
    wave_sync();
    const uint32_t v = k.L[k.l < RATE256 / 4 ? k.l : 0];
    wave_sync();
    return (int)v;
  };
  ((uint32_t *)c)[k.l] = 0;
  int w = words();
  const uint64_t signs = (uint32_t)__builtin_amdgcn_readlane(w, 0) |
                         (uint64_t)(uint32_t)__builtin_amdgcn_readlane(w, 1) << 32;
  int pos = 8, at = -1;
  for (int s = 0; s < TAU; s++) {
    const int i = N - TAU + s;
    int b;
    do {
      if (pos == RATE256) {
        keccak_f_coop(a, k);
        w = words();
        pos = 0;
      }
      b = (int)((uint32_t)__builtin_amdgcn_readlane(w, pos >> 2) >> (8 * (pos & 3)) & 0xFFu);
      pos++;
    } while (b > i);
    at = k.l == s ? b : at == b ? i : at;
  }
  wave_sync();
  if (k.l < TAU) c[at] = (int8_t)(1 - 2 * (int)(signs >> k.l & 1));
  wave_sync();
}

}  // namespace dil
