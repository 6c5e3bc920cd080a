// The word per coefficient of w that the checks of Alg. 2 take, and the hint
// computed from it.  Written without device intrinsics, so that a host test can
// compare it with Decompose over all of [0, q).
//
// A word holds (HighBits, x) with r ~ HighBits 2 gamma2 + x (mod q); after
// pack_low x is LowBits(r), and subtracting c s2 from x leaves the high bits in
// place.  For |x| < gamma2 the pair is the decomposition of the number that it
// stands for, so as long as |c s2| <= beta
//   |LowBits(w - c s2)| < gamma2 - beta  if and only if  |x - c s2| < gamma2 - beta,
// and then w - c s2 keeps w's high bits.  KeyGen's keys have |c s2| <= beta.  A key
// row may encode larger coefficients (the eta fields 5 .. 7 of three bits, 9 .. 15
// of four): there x can leave the interval by more than beta, which low_beyond
// tells, and low_carry then moves it into the next one.
//
// Adding c t0 (|c t0| < gamma2) to a low part that has passed gives u with |u| < 2
// gamma2, and the high bits change if and only if u leaves (-gamma2, gamma2]; the
// one exception is u = -gamma2 with high bits 0, which Decompose maps to 0 again
// (r = q - gamma2).
#pragma once
#include "batch_sched.h"  // DIL_HD

namespace dil {

constexpr int LOW_SHIFT = 6;  // bits of HighBits: below 44 or 16
DIL_HD int32_t pack_low(int32_t r1, int32_t r0) { return r0 * (1 << LOW_SHIFT) + r1; }
DIL_HD int32_t low_part(int32_t w) { return w >> LOW_SHIFT; }
DIL_HD int32_t low_high(int32_t w) { return w & ((1 << LOW_SHIFT) - 1); }

// |x| >= gamma2 - beta; |x| > gamma2 + beta
template <int32_t G2, int32_t BETA>
DIL_HD bool low_fails(int32_t w) { return (uint32_t)(low_part(w) + (G2 - BETA - 1)) > 2u * (G2 - BETA - 1); }
template <int32_t G2, int32_t BETA>
DIL_HD bool low_beyond(int32_t w) { return (uint32_t)(low_part(w) + G2 + BETA) > 2u * (G2 + BETA); }
// the decomposition of the number a word stands for, |x| < 2 gamma2; M = (q - 1) / (2 gamma2)
// intervals, of which the last ends one below q: M 2 gamma2 = -1 (mod q)
template <int32_t G2, int32_t M>
DIL_HD int32_t low_carry(int32_t w) {
  const int32_t x = low_part(w), r1 = low_high(w);
  if (x > G2) return r1 == M - 1 ? pack_low(0, x - 2 * G2 - 1) : pack_low(r1 + 1, x - 2 * G2);
  if (x < -G2 || (x == -G2 && r1 != 0)) return r1 == 0 ? pack_low(M - 1, x + 2 * G2 + 1) : pack_low(r1 - 1, x + 2 * G2);
  return w;
}
template <int32_t G2>
DIL_HD bool hint_of(int32_t u, int32_t high) { return u > G2 || u - (high != 0) < -G2; }

}  // namespace dil
