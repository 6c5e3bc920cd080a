// Host check of the low parts of w (paper_2211_12265_amd/csrc/lowbits.h), built with
// AddressSanitizer and UndefinedBehaviorSanitizer by tests/test_host_low_bits.py: for
// every r in [0, q), the word of r moved by d and carried is the decomposition of r + d
// by its definition; and the hint from a word is HighBits(r + u) != HighBits(r).
#include <stdint.h>
#include <stdio.h>

#include <initializer_list>

#include "lowbits.h"

using namespace dil;

static constexpr int64_t Q = 8380417;

// Decompose by definition: r0 = r mod+- alpha, and r - r0 = q - 1 becomes (0, r0 - 1)
template <int32_t G2>
static void decomp(int64_t r, int32_t &r1, int32_t &r0) {
  const int64_t alpha = 2 * G2, rp = ((r % Q) + Q) % Q;
  int64_t lo = rp % alpha;
  if (lo > G2) lo -= alpha;
  if (rp - lo == Q - 1) {
    r1 = 0;
    r0 = (int32_t)lo - 1;
  } else {
    r1 = (int32_t)((rp - lo) / alpha);
    r0 = (int32_t)lo;
  }
}

template <int32_t G2, int32_t BETA>
static int run(int most) {
  constexpr int32_t M = (int32_t)((Q - 1) / (2 * G2));
  const int32_t moves[] = {0, 1, -1, BETA, -BETA, BETA + 1, -BETA - 1, most, -most};
  long beyond = 0;
  for (int64_t r = 0; r < Q; r++) {
    int32_t r1, r0, a1, a0;
    decomp<G2>(r, r1, r0);
    const int32_t w = pack_low(r1, r0);
    if (low_part(w) != r0 || low_high(w) != r1) return fprintf(stderr, "packing of %ld\n", (long)r), 1;
    for (int32_t d : moves) {
      const int32_t v = w + d * (1 << LOW_SHIFT), c = low_carry<G2, M>(v);
      decomp<G2>(r + d, a1, a0);
      if (low_part(c) != a0 || low_high(c) != a1) return fprintf(stderr, "%ld moved by %d\n", (long)r, d), 1;
      // a word that low_beyond does not name passes the bound as it is or not at all, and keeps its high bits
      const bool pass = a0 < G2 - BETA && a0 > -(G2 - BETA), plain = !low_fails<G2, BETA>(v);
      if (pass == low_fails<G2, BETA>(c)) return fprintf(stderr, "norm of %ld moved by %d\n", (long)r, d), 1;
      if (!low_beyond<G2, BETA>(v) && (pass != plain || (pass && c != v)))
        return fprintf(stderr, "bound at %ld moved by %d\n", (long)r, d), 1;
      beyond += low_beyond<G2, BETA>(v);
    }
    if (r0 < G2 - BETA && r0 > -(G2 - BETA))
      for (int32_t u : {1, G2 - 1, -(G2 - 1), G2 - r0, G2 - r0 + 1, -G2 - r0, -G2 - r0 - 1}) {
        if (u >= G2 || u <= -G2) continue;
        decomp<G2>(r + u, a1, a0);
        if (hint_of<G2>(low_part(w) + u, low_high(w)) != (a1 != r1))
          return fprintf(stderr, "hint of %ld and %d\n", (long)r, u), 1;
      }
  }
  printf("ok M=%d beyond=%ld\n", M, beyond);
  return beyond == 0;
}

// most: tau times the largest magnitude that an eta field encodes
int main() { return run<95232, 78>(39 * 5) || run<261888, 196>(49 * 11) || run<261888, 120>(60 * 5); }
