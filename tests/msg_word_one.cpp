// Host check of the word-at-a-time form of the message-representative blocks
// (mw_fetch_one / mw_word_one in paper_2211_12265_amd/csrc/msg_words.h), built
// with AddressSanitizer and UndefinedBehaviorSanitizer by
// tests/test_host_msg_words_one.py: every word of every block of prefix || M ||
// padding equals the padded byte string (and so do the blocks that MwPlan::inner names, read without masks), for every misalignment and length, M
// lying in a heap buffer of exactly the dwords that cover it.
//
// usage: msg_word_one MAXLEN
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "msg_words.h"

using namespace dil;

template <int PB>
static int run(int maxlen) {
  int cases = 0;
  uint8_t prefix[PB];
  for (int i = 0; i < PB; i++) prefix[i] = i < PB / 4 * 4 ? (uint8_t)(37 * i + 11) : 0;
  for (int sh = 0; sh < 4; sh++)
    for (int len = 0; len <= maxlen; len++) {
      const int nd = len ? (sh + len + 3) / 4 : 0;
      uint32_t *buf = nd ? (uint32_t *)malloc(4 * (size_t)nd) : nullptr;
      static uint32_t none;
      uint8_t *msg = nd ? (uint8_t *)buf + sh : (uint8_t *)&none + sh;
      for (int i = 0; i < len; i++) msg[i] = (uint8_t)(i * 151 + len + 7 * sh);
      const int nblk = (PB + len) / MW_RATE + 1;
      std::vector<uint8_t> want((size_t)nblk * MW_RATE, 0);
      memcpy(want.data(), prefix, PB);
      if (len) memcpy(want.data() + PB, msg, (size_t)len);
      want[(size_t)PB + len] ^= 0x1F;
      want[want.size() - 1] ^= 0x80;
      const MwPlan<PB> pl(msg, (uint64_t)len);
      if (pl.nblk != (uint64_t)nblk) return fprintf(stderr, "blocks %d %d\n", sh, len), 1;
      for (int b = 0; b < nblk; b++)
        for (int j = 0; j < MW_WPB; j++) {
          uint32_t pre = 0, lo, hi, w;
          if (b == 0 && 4 * j + 4 <= PB) memcpy(&pre, prefix + 4 * j, 4);
          mw_fetch_one(pl, (uint64_t)b, j, lo, hi);
          w = mw_word_one(pl, (uint64_t)b, j, pre, lo, hi);
          uint32_t x;
          memcpy(&x, want.data() + (size_t)b * MW_RATE + 4 * j, 4);
          if (w != x) return fprintf(stderr, "PB %d sh %d len %d block %d word %d\n", PB, sh, len, b, j), 1;
        }
      // the blocks that are read without masks: 34 words as each lane of a pair takes them
      if (pl.inner() < 1 || pl.inner() > pl.nblk) return fprintf(stderr, "inner %d %d\n", sh, len), 1;
      for (uint64_t b = 1; b < pl.inner(); b++)
        for (int j = 0; j < MW_WPB; j++) {
          const uint32_t *p = pl.inner_words(b) + j;
          uint32_t x;
          memcpy(&x, want.data() + b * MW_RATE + 4 * j, 4);
          if (mw_funnel(p[1], p[0], pl.fs) != x) return fprintf(stderr, "inner PB %d sh %d len %d\n", PB, sh, len), 1;
        }
      free(buf);
      cases++;
    }
  printf("ok PB=%d cases=%d\n", PB, cases);
  return 0;
}

int main(int argc, char **argv) {
  const int maxlen = argc > 1 ? atoi(argv[1]) : 300;
  return run<32>(maxlen) || run<64>(maxlen) || run<66>(maxlen);
}
