// SHAKE128/256 sponges over byte sources, and the per-lane samplers
// (Sec. 2.3 "Sampling"; Alg. 1 ExpandA/ExpandS, Alg. 2 ExpandMask/SampleInBall).
// Each lane runs its own sponge (see keccak.h).
#pragma once
#include "keccak.h"
#include "poly.h"

namespace dil {

constexpr int RATE128 = 168, RATE256 = 136;

// Absorb a message of `len` bytes into a zeroed state and apply SHAKE padding
// (suffix 1111 then 10*1).  `word(pos)` must return the little-endian 8-byte
// word of message bytes [pos, pos + 8), with bytes at or beyond `len` zero.
// On return the first output block is in s[0 .. RATE/4).
template <int RATE, class W>
__device__ __forceinline__ void shake_absorb(uint32_t s[50], uint64_t len, W word) {
  keccak_zero(s);
  uint64_t nblk = len / RATE + 1;
  for (uint64_t b = 0; b < nblk; b++) {
#pragma unroll
    for (int w = 0; w < RATE / 8; w++) {
      uint64_t pos = b * RATE + 8 * w;
      uint64_t v = pos < len ? word(pos) : 0;
      if (pos <= len && len < pos + 8) v ^= (uint64_t)0x1F << (8 * (len - pos));
      if (w == RATE / 8 - 1 && b == nblk - 1) v ^= (uint64_t)0x80 << 56;
      s[2 * w] ^= (uint32_t)v;
      s[2 * w + 1] ^= (uint32_t)(v >> 32);
    }
    keccak_f(s);
  }
}

// ---- single-block absorption of the short fixed-size sampler seeds ----
// seed = 32-byte rho (word source) || two nonce bytes, SHAKE128
template <class W>
__device__ __forceinline__ void absorb_seed34(uint32_t s[50], W rho_word, uint32_t nonce16) {
  keccak_zero(s);
#pragma unroll
  for (int w = 0; w < 4; w++) {
    uint64_t v = rho_word(8 * w);
    s[2 * w] = (uint32_t)v;
    s[2 * w + 1] = (uint32_t)(v >> 32);
  }
  s[8] = nonce16 | (0x1Fu << 16);
  s[2 * (RATE128 / 8 - 1) + 1] ^= 0x80u << 24;
  keccak_f(s);
}
// seed = 64-byte rho' (8-byte aligned) || LE16 nonce, SHAKE256
__device__ __forceinline__ void absorb_seed66(uint32_t s[50], const uint8_t *rhop, uint32_t nonce16) {
  keccak_zero(s);
  const uint64_t *rp = (const uint64_t *)rhop;
#pragma unroll
  for (int w = 0; w < 8; w++) {
    uint64_t v = rp[w];
    s[2 * w] = (uint32_t)v;
    s[2 * w + 1] = (uint32_t)(v >> 32);
  }
  s[16] = (nonce16 & 0xFFFFu) | (0x1Fu << 16);
  s[2 * (RATE256 / 8 - 1) + 1] ^= 0x80u << 24;
  keccak_f(s);
}

// ExpandMask: the lane's SHAKE256 stream (absorbed and permuted once) stored as
// it comes, 16 bytes at a time.  The first 32 B bytes are the B-bit little-endian
// fields v of the polynomial's 256 coefficients gamma1 - v, which the readers
// unpack (load_mask): 576 / 640 bytes per polynomial move instead of 1024, and
// the squeezing lane does no work per coefficient.  out is 16-byte aligned.
template <int B>
__device__ __forceinline__ void expand_mask_squeeze(uint32_t s[50], uint8_t *out) {
  constexpr int WPB = RATE256 / 4;              // 34 words per block
  constexpr int NWORD = N * B / 32;             // 144 / 160
  constexpr int NBLK = (NWORD + WPB - 1) / WPB; // 5
  uint32_t quad[4];
#pragma unroll
  for (int blk = 0; blk < NBLK; blk++) {
    if (blk > 0) keccak_f(s);
#pragma unroll
    for (int w = 0; w < WPB; w++) {
      const int gw = blk * WPB + w;
      if (gw < NWORD) {
        quad[gw & 3] = s[w];
        if ((gw & 3) == 3) ((uint4 *)out)[gw >> 2] = make_uint4(quad[0], quad[1], quad[2], quad[3]);
      }
    }
  }
}
// the lane's strided coefficients (t + 16 r) of a polynomial stored by
// expand_mask_squeeze: field t + 16 r starts 16 B r bits, a whole number of
// words, after field t.  Every field is fetched as the two words it may span;
// the second word of a row's last field is the one after the row (its bits are
// not used), so a row is followed by at least four more bytes of its memory.
// TOGETHER: all words are requested before the first field is cut out.  Left alone, in
// kernels near their register limit the compiler waits for each pair of words before
// it requests the next (loop kernel, 10,000 tasks of levels 2 / 3 / 5, mean of six
// batches: 1212 / 2188 / 2242 us, with it 1045 / 1880 / 1920; where the registers leave
// room, as in rd_w_k, it asks for them early enough by itself).
template <int B, int32_t GAMMA1, bool TOGETHER = false>
__device__ __forceinline__ void load_mask(int32_t x[16], const uint8_t *row, int t) {
  const uint32_t *w = (const uint32_t *)row + ((B * t) >> 5);
  const int sh = (B * t) & 31;
  uint32_t lo[16], hi[16];
#pragma unroll
  for (int r = 0; r < 16; r++) {
    lo[r] = w[r * (B / 2)];
    hi[r] = w[r * (B / 2) + 1];
  }
  if constexpr (TOGETHER) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = GAMMA1 - (int32_t)(__builtin_amdgcn_alignbit(hi[r], lo[r], sh) & ((1u << B) - 1u));
}

// ExpandS: the lane's SHAKE256 stream (absorbed and permuted once) stored as it
// comes, S_POLY bytes apart: two blocks, or as many as hold 256 accepted nibbles
// (eta = 2: v < 15, eta = 4: v < 9).  The readers pick them out (dev_collect_s):
// one lane that tests 544 nibbles one after another and stores 256 words of its
// own takes five times as long as its two permutations.  Two blocks are short of
// 256 in one polynomial of 10^5 (eta = 4), four in fewer than one of 10^100.
constexpr int S_BLOCKS = 4, S_POLY = S_BLOCKS * RATE256;
static_assert(S_POLY % 16 == 0, "read 16 bytes at a time");
// bit 0 of every accepted nibble of w
template <int ETA>
__device__ __forceinline__ uint32_t s_accepted(uint32_t w) {
  const uint32_t r = ETA == 2 ? w & (w >> 1) & (w >> 2) & (w >> 3) : (w >> 3) & (w | (w >> 1) | (w >> 2));
  return ~r & 0x11111111u;
}
template <int ETA>
__device__ __forceinline__ void expand_s_squeeze(uint32_t s[50], uint8_t *out) {
  int got = 0;
#pragma unroll 1
  for (int blk = 0;; blk++) {
    uint64_t *o = (uint64_t *)(out + blk * RATE256);
#pragma unroll
    for (int w = 0; w < RATE256 / 8; w++) o[w] = (uint64_t)s[2 * w + 1] << 32 | s[2 * w];
#pragma unroll
    for (int w = 0; w < RATE256 / 4; w++) got += __popc(s_accepted<ETA>(s[w]));
    if (blk + 1 == S_BLOCKS || (blk > 0 && got >= N)) break;
    keccak_f(s);
  }
}

}  // namespace dil
