// Keccak-f[1600] with one state on a 16-lane DPP row, for hash chains that have
// the chip to themselves (small batches, the last rounds of Sign): what counts
// there is the length of one permutation, and a lone wavefront issues one
// instruction per five cycles whatever its lanes hold.
//
// Lane l of the row holds half h = l & 1 (low / high 32 bits) of the words of
// sheet x = (l mod 10) / 2, register y the word (x, y); lanes 10 .. 15 repeat
// x = 0, 1, 2, so that neighbouring sheets are a lane shift away:
//   theta  column parity in the lane, C[x - 1] and C[x + 1] from lanes l -+ 2
//          (lanes 10, 11 take C[1] from lanes 2, 3), the rotation's other half
//          from the neighbour lane;
//   rho, pi  the five words go through LDS: every lane reads back, for its new
//          place, the two halves in the order in which one v_alignbit with the
//          word's own amount rotates them;
//   chi    the next two sheets from lanes l + 2, l + 4.
// After chi lanes 0 .. 11 are valid, after theta lanes 2 .. 11, which hold every
// sheet once and are the ones whose words are kept; the read-back makes all 16
// valid again.  34 VALU and 14 LDS instructions per round against 120 VALU on a
// lane pair (keccak_pair.h): 3.4 times the issue slots per state, half the time
// per permutation of a lone wavefront (3.1 against 6.8 us): the mu chains of 2,503
// messages of up to 4 KB 328 -> 176 us.  4,096 states take 4.4 us per permutation,
// 8,192 5.6, 10,240 6.8, where 320 wavefronts of pairs need no longer.  Round
// constants from scalar loads instead of LDS: 3.8 us alone, 5.1 with 4,096 states.
//
// The functions after the two engines run on either (E: RowKeccak or
// WaveKeccak, keccak_wave.h).
#pragma once
#include "keccak_wave.h"
#include "kernels.h"

namespace dil {

template <int Y>
struct RowRot {
  static constexpr uint32_t v = row_rot(Y);
};

// the lane's constants; L: the wavefront's KECCAK_LDS words: four states of 50
// words, ROW_ST apart, so that the accesses of two rows hit different banks, and
// a dump for unkept words
constexpr int ROW_ST = 54;
struct RowKeccak {
  static constexpr int NR = 5, NA = 4, ND = 2;  // registers; those with words of the rate; with words 0 .. 9
  static constexpr int LANES = 16, STATES = 4;
  uint32_t *L;
  int x, h, l;
  bool own;             // holds words of its own (lanes 10 .. 15 are copies)
  int st;               // the state's words in L
  int wr;               // where the lane keeps word (x, 0); (x, y) is 10 y further
  int p[5], q[5];       // high and low operand of the rotation that yields word (x, y)
  uint32_t s[5];        // its amount
  const uint32_t *rc;   // round constants
  __device__ __forceinline__ RowKeccak(uint32_t *lds, int lane) {
    L = lds;
    l = lane & 15;
    const int m = l < 10 ? l : l - 10;
    own = l < 10;
    x = m >> 1;
    h = m & 1;
    st = ROW_ST * ((lane >> 4) & 3);
    wr = l >= 2 && l < 12 ? st + 2 * x + h : 4 * ROW_ST - 4;
    place<0>();
    place<1>();
    place<2>();
    place<3>();
    place<4>();
    rc = kc_rc_lds<LANES>(L, l, x == 0, h);
  }
  // where register Y is read from: word (sx, sy) with (x, Y) = (sy, 2 sx + 3 sy)
  template <int Y>
  __device__ __forceinline__ void place() {
    int sx = (3 * Y) % 5 + x;
    sx = sx >= 5 ? sx - 5 : sx;
    const int n = (int)((RowRot<Y>::v >> (6 * x)) & 63u);
    const int mine = st + 2 * (sx + 5 * x) + h, other = mine + 1 - 2 * h;
    p[Y] = n > 32 ? other : mine;
    q[Y] = n == 0 || n > 32 ? mine : other;
    s[Y] = (uint32_t)-n & 31u;  // 32 - n, 64 - n, or 0
  }
  // 8-byte word index of register y, and the 32-bit word of it that this lane holds
  __device__ __forceinline__ int word(int y) const { return 5 * y + x; }
  __device__ __forceinline__ int half_word(int y) const { return 2 * word(y) + h; }
  // whether `v` holds on a lane of the state
  __device__ __forceinline__ bool any(bool v) const { return (__ballot(v) >> (st / ROW_ST * 16) & 0xFFFFu) != 0; }
};

__device__ __forceinline__ void keccak_f_coop(uint32_t a[5], const RowKeccak &k) {
  const uint32_t *rc = k.rc;
#pragma unroll 4
  for (int ir = 0; ir < 24; ir++) {
    const uint32_t rcv = rc[0];
    rc += 2;
    const uint32_t c = xor3(xor3(a[0], a[1], a[2]), a[3], a[4]);
    uint32_t cm;
    const uint32_t r = row_theta(c, cm);
#pragma unroll
    for (int y = 0; y < 5; y++) k.L[k.wr + 10 * y] = xor3(a[y], cm, r);
    wave_sync();
    uint32_t b[5];
#pragma unroll
    for (int y = 0; y < 5; y++) b[y] = __builtin_amdgcn_alignbit(k.L[k.p[y]], k.L[k.q[y]], k.s[y]);
    wave_sync();
#pragma unroll
    for (int y = 0; y < 5; y++) a[y] = chi3(b[y], row_dpp<0x102>(b[y]), row_dpp<0x104>(b[y]));
    a[0] ^= rcv;
  }
}

// SHAKE256 absorption of a LEN-byte string (LEN a multiple of 8) given by its
// 32-bit words: word(i) is called for 4 i < LEN only.  The next block's words
// are requested before the current one is permuted.
template <int LEN, class E, class W>
__device__ __forceinline__ void shake256_absorb_coop(uint32_t a[E::NR], const E &k, W word) {
  static_assert(LEN % 8 == 0, "whole 8-byte words");
  constexpr int RATE = 136, NBLK = LEN / RATE + 1;
  auto fetch = [&](uint32_t v[E::NA], int blk) {
#pragma unroll
    for (int y = 0; y < E::NA; y++) {
      const int w = k.word(y), pos = blk * RATE + 8 * w;
      v[y] = w < RATE / 8 && pos < LEN ? word(blk * (RATE / 4) + k.half_word(y)) : 0u;
      if (w < RATE / 8 && pos == LEN && !k.h) v[y] = 0x1Fu;                     // suffix 1111 + first pad bit
      if (w == RATE / 8 - 1 && blk == NBLK - 1 && k.h) v[y] ^= 0x80u << 24;     // last pad bit
    }
  };
#pragma unroll
  for (int y = 0; y < E::NR; y++) a[y] = 0;
  uint32_t v[E::NA];
  fetch(v, 0);
#pragma unroll 1
  for (int blk = 0; blk < NBLK; blk++) {
#pragma unroll
    for (int y = 0; y < E::NA; y++) a[y] ^= v[y];
    if (blk + 1 < NBLK) fetch(v, blk + 1);
    keccak_f_coop(a, k);
  }
}

// SHAKE256 absorption of X = prefix || M (msg_words.h): pre[y] is the lane's
// prefix word of register y where word(y) < PB / 8.
template <int PB, class E>
__device__ __forceinline__ void absorb_prefix_msg_coop(uint32_t a[E::NR], const E &k, const uint32_t pre[E::ND],
                                                      const uint8_t *msg, uint64_t mlen) {
  using Plan = MwPlan<PB>;
  const Plan pl(msg, mlen);
  uint32_t lo[E::NA], hi[E::NA];
  auto fetch = [&](uint64_t blk) {
#pragma unroll
    for (int y = 0; y < E::NA; y++) {
      lo[y] = hi[y] = 0;
      if (k.word(y) < MW_RATE / 8) mw_fetch_one(pl, blk, k.half_word(y), lo[y], hi[y]);
    }
  };
  const uint32_t p0 = pre[0], p1 = pre[E::ND - 1];
#pragma unroll
  for (int y = 0; y < E::NR; y++) a[y] = 0;
  fetch(0);
  for (uint64_t blk = 0; blk < pl.nblk; blk++) {
#pragma unroll
    for (int y = 0; y < E::NA; y++)
      if (k.word(y) < MW_RATE / 8)
        a[y] ^= mw_word_one(pl, blk, k.half_word(y), y == 0 ? p0 : p1, lo[y], hi[y]);
    if (blk + 1 < pl.nblk) fetch(blk + 1);
    keccak_f_coop(a, k);
  }
}

// SampleInBall on a row whose state holds the first SHAKE256 block of ctilde;
// c: 256 bytes, bw: 34 words (the wavefront form needs none), both LDS, 4-byte
// aligned.  As on a wavefront, lane l follows the signs of steps l, l + 16, ...;
// the rows take one byte each per step, whether they keep it or not, so that the
// bytes are read ahead, four at a time.  (With the array in LDS a step waited for
// the byte and for c[b]: the challenges of 8,192 candidates 64 us.)
template <int TAU>
__device__ __forceinline__ void sample_in_ball_coop(uint32_t a[5], const RowKeccak &k, int8_t *c, uint32_t *bw) {
  constexpr int SLOTS = (TAU + 15) / 16;
  auto stage = [&]() {
    if (k.own) {
#pragma unroll
      for (int y = 0; y < RowKeccak::NA; y++)
        if (k.word(y) < RATE256 / 8) bw[k.half_word(y)] = a[y];
    }
    wave_sync();
  };
  stage();
  uint32_t *cw = (uint32_t *)c;
#pragma unroll
  for (int w = 0; w < N / 64; w++) cw[16 * w + k.l] = 0;
  const uint64_t signs = (uint64_t)bw[0] | ((uint64_t)bw[1] << 32);
  int at[SLOTS], i = N - TAU;
#pragma unroll
  for (int q = 0; q < SLOTS; q++) at[q] = -1;
  for (int w = 2;; w++) {
    if (w == RATE256 / 4) {
      wave_sync();
      keccak_f_coop(a, k);
      stage();
      w = 0;
    }
    const uint32_t v = bw[w];
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int b = (int)((v >> (8 * j)) & 0xFFu);
      const bool keep = b <= i && i < N;
      const int from = keep ? b : N, step = keep ? i - (N - TAU) : N;
#pragma unroll
      for (int q = 0; q < SLOTS; q++) at[q] = step == 16 * q + k.l ? b : at[q] == from ? i : at[q];
      i += keep;
    }
    if (!wave_any(i < N)) break;
  }
  wave_sync();
#pragma unroll
  for (int q = 0; q < SLOTS; q++)
    if (16 * q + k.l < TAU) c[at[q]] = (int8_t)(1 - 2 * (int)(signs >> (16 * q + k.l) & 1));
  wave_sync();
}

// ctilde = H(mu || w1) and c = SampleInBall(ctilde) (as dev_challenge_pair); ctilde_out: CT / 4 words
template <int LV, class E>
__device__ __forceinline__ void dev_challenge_coop(const uint8_t *mu, const uint8_t *w1, const E &k,
                                                   uint32_t *ctilde_out, int8_t *c, uint32_t *bw) {
  constexpr int CW = P<LV>::CT / 8;  // 8-byte words of ctilde
  uint32_t a[E::NR];
  shake256_absorb_coop<P<LV>::MUW1>(a, k, [&](int i) {
    return i < 16 ? ((const uint32_t *)mu)[i] : ((const uint32_t *)w1)[i - 16];
  });
#pragma unroll
  for (int y = 0; y < E::NR; y++) {
    const int w = k.word(y);
    if (w < CW) {
      if (k.own) ctilde_out[k.half_word(y)] = a[y];
    } else {
      a[y] = w == CW && !k.h ? 0x1Fu : 0u;
    }
    if (w == RATE256 / 8 - 1 && k.h) a[y] ^= 0x80u << 24;
  }
  keccak_f_coop(a, k);
  sample_in_ball_coop<Lv<LV>::TAU>(a, k, c, bw);
}

// as dev_prep_pair (kernels.h)
template <int LV, bool INTERNAL, class E>
__device__ __forceinline__ void dev_prep_coop(uint32_t t, const E &k, const uint8_t *sk, const uint32_t *key_idx, const uint8_t *msg, const uint64_t *msg_off,
                                             const uint8_t *rnd, const Ws &ws, uint32_t *err) {
  const size_t key = key_idx ? key_idx[t] : t;
  const uint32_t *skw = (const uint32_t *)(sk + key * P<LV>::SK);
  const uint64_t o0 = msg_off[t], o1 = msg_off[t + 1];
  uint64_t mlen = 0;
  if (o1 >= o0) mlen = o1 - o0;
  else if (k.l == 0) atomicOr(err, 1u);  // decreasing msg_off: message treated as empty
  uint32_t pre[E::ND];
#pragma unroll
  for (int y = 0; y < E::ND; y++) pre[y] = k.word(y) < P<LV>::TRB / 8 ? skw[16 + k.half_word(y)] : 0u;
  uint32_t a[E::NR];
  absorb_prefix_msg_coop<mu_prefix_bytes<LV, INTERNAL>()>(a, k, pre, msg + o0, mlen);
  uint32_t *muw = (uint32_t *)(ws.muw1 + (size_t)t * muw1_stride<LV>());
  uint32_t *rp = (uint32_t *)(ws.rhop + (size_t)t * 64);
  // mu also to LDS, from where it is absorbed at another place
#pragma unroll
  for (int y = 0; y < E::ND; y++)
    if (k.own && k.word(y) < 8) {
      muw[k.half_word(y)] = a[y];
      k.L[k.st + k.half_word(y)] = a[y];
    }
  wave_sync();
  const bool round3_rnd = !Lv<LV>::MLDSA && rnd;  // rho' is the task's rnd itself
  constexpr int MU0 = Lv<LV>::MLDSA ? 8 : 4;      // word of mu in K || rnd || mu, K || mu
  uint32_t b[E::NR];
#pragma unroll
  for (int y = 0; y < E::NR; y++) {
    const int w = k.word(y), i = k.half_word(y);
    b[y] = 0;
    if (w < 4) b[y] = skw[8 + i];
    else if (w < MU0) b[y] = rnd ? ((const uint32_t *)(rnd + (size_t)t * 32))[i - 8] : 0u;
    else if (w < MU0 + 8) b[y] = k.L[k.st + i - 2 * MU0];
    if (w == MU0 + 8 && !k.h) b[y] ^= 0x1Fu;
    if (w == RATE256 / 8 - 1 && k.h) b[y] ^= 0x80u << 24;
  }
  wave_sync();
  if (!round3_rnd) keccak_f_coop(b, k);
#pragma unroll
  for (int y = 0; y < E::ND; y++)
    if (k.own && k.word(y) < 8)
      rp[k.half_word(y)] = round3_rnd ? ((const uint32_t *)(rnd + (size_t)t * 64))[k.half_word(y)] : b[y];
  if (k.l == 0) {
    ws.kappa[t] = 0;
    ws.active0[t] = t;
  }
}

// as dev_hash_pair
template <int LV, bool INTERNAL, class E>
__device__ __forceinline__ void dev_hash_coop(uint32_t t, const E &k, const uint8_t *pk, const uint32_t *key_idx,
                                              const uint8_t *msg, const uint64_t *msg_off, const Ws &ws,
                                              uint32_t *err) {
  using PP = P<LV>;
  const size_t key = key_idx ? key_idx[t] : t;
  uint32_t a[E::NR], pre[E::ND];
  if (ws.tr) {
    const uint32_t *tg = (const uint32_t *)(ws.tr + key * PP::TRB);
#pragma unroll
    for (int y = 0; y < E::ND; y++) pre[y] = k.word(y) < PP::TRB / 8 ? tg[k.half_word(y)] : 0u;
  } else {
    const uint32_t *pkr = (const uint32_t *)(pk + key * PP::PK);
    shake256_absorb_coop<PP::PK>(a, k, [&](int i) { return pkr[i]; });
    // the lane's words of the digest are its words of the prefix
#pragma unroll
    for (int y = 0; y < E::ND; y++) pre[y] = a[y];
  }
  const uint64_t o0 = msg_off[t], o1 = msg_off[t + 1];
  uint64_t mlen = 0;
  if (o1 >= o0) mlen = o1 - o0;
  else if (k.l == 0) atomicOr(err, 1u);  // decreasing msg_off: message treated as empty
  absorb_prefix_msg_coop<mu_prefix_bytes<LV, INTERNAL>()>(a, k, pre, msg + o0, mlen);
  uint32_t *muw = (uint32_t *)(ws.muw1 + (size_t)t * muw1_stride<LV>());
#pragma unroll
  for (int y = 0; y < E::ND; y++)
    if (k.own && k.word(y) < 8) muw[k.half_word(y)] = a[y];
}

// c = SampleInBall(ctilde) of task t
template <int LV, class E>
__device__ __forceinline__ void dev_ball_coop(const uint8_t *ctilde, const E &k, int8_t *c, uint32_t *bw) {
  uint32_t a[E::NR];
#pragma unroll
  for (int y = 0; y < E::NR; y++) {
    const int w = k.word(y);
    a[y] = w < P<LV>::CT / 8 ? (uint32_t)load_le_bytes(ctilde + 4 * k.half_word(y), 4) : w == P<LV>::CT / 8 && !k.h ? 0x1Fu : 0u;
    if (w == RATE256 / 8 - 1 && k.h) a[y] ^= 0x80u << 24;
  }
  keccak_f_coop(a, k);
  sample_in_ball_coop<Lv<LV>::TAU>(a, k, c, bw);
}
// the dense challenge from LDS to a 16-byte aligned global row
template <class E>
__device__ __forceinline__ void store_c_coop(const int8_t *c, int8_t *dst, const E &k) {
  wave_sync();
  if constexpr (E::LANES == 64) {
    ((uint32_t *)dst)[k.l] = ((const uint32_t *)c)[k.l];
  } else {
    const uint32_t *cw = (const uint32_t *)c + 4 * k.l;
    ((int4 *)dst)[k.l] = make_int4(cw[0], cw[1], cw[2], cw[3]);
  }
}

// ---- kernels: one-wavefront workgroups of 32 lane pairs, four rows or one state ----
// mu needs one permutation per 136 message bytes in series, whatever the chip
// does beside it: up to 31 for 4 KB, and Verify's tr = H(pk) 10 / 15 / 20 before
// them.  A batch that leaves room gives every task a row or a wavefront.  Larger
// ones take lane pairs: beside ExpandA rows would cost it more than they gain
// (level-3 Verify, 10,000 tasks of up to 4 KB: 555-697 us with rows for the
// messages of more than 2 KB against 551).
constexpr uint32_t ROW_STATES = 4096, ROW_ALONE = 8192;  // beside ExpandA; with the chip to themselves
#define DIL_COOP_TASK(E)                                           \
  __shared__ uint32_t L[KECCAK_LDS];                               \
  __builtin_amdgcn_s_setprio(3);                                   \
  const uint32_t t = blockIdx.x * E::STATES + threadIdx.x / E::LANES; \
  if (t >= count) return; /* a whole state */                      \
  const E k(L, threadIdx.x);

template <int LV, bool INTERNAL>
__global__ void __launch_bounds__(64) sg_prep_k(const uint8_t *sk, const uint32_t *key_idx,
                                                    const uint8_t *msg, const uint64_t *msg_off, const uint8_t *rnd, Ws ws, uint32_t count, uint32_t *err) {
  __builtin_amdgcn_s_setprio(3);  // long dependent chains beside ExpandA: these waves issue first
  const uint32_t t = blockIdx.x * 32 + (threadIdx.x >> 1);
  if (t < count) dev_prep_pair<LV, INTERNAL>(t, threadIdx.x & 1, sk, key_idx, msg, msg_off, rnd, ws, err);
}
template <int LV, bool INTERNAL, class E>
__global__ void __launch_bounds__(64) sg_prep_coop_k(const uint8_t *sk, const uint32_t *key_idx,
                                                    const uint8_t *msg, const uint64_t *msg_off, const uint8_t *rnd, Ws ws, uint32_t count, uint32_t *err) {
  DIL_COOP_TASK(E)
  dev_prep_coop<LV, INTERNAL>(t, k, sk, key_idx, msg, msg_off, rnd, ws, err);
}
template <int LV, bool INTERNAL>
__global__ void __launch_bounds__(64) vf_hash_k(const uint8_t *pk, const uint32_t *key_idx,
                                                    const uint8_t *msg, const uint64_t *msg_off, Ws ws, uint32_t count, uint32_t *err) {
  __builtin_amdgcn_s_setprio(3);  // long dependent chains beside ExpandA: these waves issue first
  const uint32_t t = blockIdx.x * 32 + (threadIdx.x >> 1);
  if (t < count) dev_hash_pair<LV, INTERNAL>(t, threadIdx.x & 1, pk, key_idx, msg, msg_off, ws, err);
}
template <int LV, bool INTERNAL, class E>
__global__ void __launch_bounds__(64) vf_hash_coop_k(const uint8_t *pk, const uint32_t *key_idx,
                                                    const uint8_t *msg, const uint64_t *msg_off, Ws ws, uint32_t count, uint32_t *err) {
  DIL_COOP_TASK(E)
  dev_hash_coop<LV, INTERNAL>(t, k, pk, key_idx, msg, msg_off, ws, err);
}

// as vf_prep_k
template <int LV, class E>
__global__ void __launch_bounds__(64) vf_prep_coop_k(const uint8_t *sig, Ws ws, uint32_t count) {
  __shared__ __align__(16) int8_t cl[E::STATES][C_ROW];
  __shared__ uint32_t bb[E::STATES][RATE256 / 4];
  DIL_COOP_TASK(E)
  const int p = threadIdx.x / E::LANES;
  dev_ball_coop<LV>(sig + (size_t)t * P<LV>::SIG, k, cl[p], bb[p]);
  store_c_coop(cl[p], ws.cpoly + (size_t)t * N, k);
}
// The fronts of a small Verify that has its tables: workgroups 0 .. count - 1 hash
// mu, the others sample the challenge and do the main part, a wavefront each.  In
// one launch because the hash chain, 45 permutations for 6 KB, leaves the chip
// nearly idle: 333 messages at ML-DSA-87 took 155 us with three launches
// in series, 128 with one (one card; the call varies between 110 and 190).
constexpr uint32_t FRONT_TASKS = WAVE_STATES / 2;  // above, the two would queue for LDS
template <int LV, bool INTERNAL>
__global__ void __launch_bounds__(64, 3)
    vf_front_k(const uint8_t *pk, const uint32_t *key_idx, const uint8_t *msg, const uint64_t *msg_off,
               const uint8_t *sig, Ws ws, uint32_t count, uint32_t *err) {
  __shared__ VfLds<LV> lds;
  static_assert(sizeof lds.zh >= 4 * KECCAK_LDS && sizeof lds.region >= N, "the sponge's words, the challenge");
  const int lane = threadIdx.x;
  const WaveKeccak k((uint32_t *)lds.zh, lane);
  if (blockIdx.x < count) {
    __builtin_amdgcn_s_setprio(3);
    dev_hash_coop<LV, INTERNAL>(blockIdx.x, k, pk, key_idx, msg, msg_off, ws, err);
    return;
  }
  const uint32_t task = blockIdx.x - count;
  dev_ball_coop<LV>(sig + (size_t)task * P<LV>::SIG, k, (int8_t *)lds.region, nullptr);
  const uint32_t cw = lds.region[lane];
  wave_sync();
  dev_vf_main<LV>(task, cw, lds, pk, key_idx, sig, ws);
}

// as vf_final_k
template <int LV, class E>
__global__ void __launch_bounds__(64) vf_final_coop_k(const uint8_t *sig, Ws ws, int32_t *verdict, uint32_t count) {
  DIL_COOP_TASK(E)
  const uint32_t *row = (const uint32_t *)(ws.muw1 + (size_t)t * muw1_stride<LV>());
  uint32_t a[E::NR];
  shake256_absorb_coop<P<LV>::MUW1>(a, k, [&](int i) { return row[i]; });
  const uint8_t *sg = sig + (size_t)t * P<LV>::SIG;
  bool diff = false;
#pragma unroll
  for (int y = 0; y < E::ND; y++)
    if (k.own && k.word(y) < P<LV>::CT / 8) diff |= (uint32_t)load_le_bytes(sg + 4 * k.half_word(y), 4) != a[y];
  diff = k.any(diff);
  if (k.l == 0) verdict[t] = (ws.flag[t] && !diff) ? 1 : 0;
}

// as sg_chal_k
template <int LV, class E>
__global__ void __launch_bounds__(64) sg_chal_coop_k(Ws ws, const uint32_t *active, uint32_t count) {
  __shared__ __align__(16) int8_t cl[E::STATES][C_ROW];
  __shared__ uint32_t bb[E::STATES][RATE256 / 4];
  DIL_COOP_TASK(E)
  const int p = threadIdx.x / E::LANES;
  const uint32_t task = active[t];
  const uint8_t *row = ws.muw1 + (size_t)task * muw1_stride<LV>();
  dev_challenge_coop<LV>(row, row + 64, k, (uint32_t *)(ws.ctilde + (size_t)task * CT_STRIDE), cl[p], bb[p]);
  store_c_coop(cl[p], ws.cpoly + (size_t)task * N, k);
}

// tr = H(pk) (TRB bytes) to out rows, one state per key
template <int LV, class E>
__global__ void __launch_bounds__(64) tr_coop_k(const uint8_t *pk, uint8_t *out, size_t out_stride, uint32_t count) {
  DIL_COOP_TASK(E)
  const uint32_t *p = (const uint32_t *)(pk + (size_t)t * P<LV>::PK);
  uint32_t a[E::NR];
  shake256_absorb_coop<P<LV>::PK>(a, k, [&](int i) { return p[i]; });
  uint32_t *o = (uint32_t *)(out + (size_t)t * out_stride);
#pragma unroll
  for (int y = 0; y < E::ND; y++)
    if (k.own && k.word(y) < P<LV>::TRB / 8) o[k.half_word(y)] = a[y];
}
// the same on a lane pair, for batches that fill the chip
template <int LV>
__global__ void __launch_bounds__(64) tr_pair_k(const uint8_t *pk, uint8_t *out, size_t out_stride, uint32_t count) {
  const uint32_t t = (blockIdx.x * 64 + threadIdx.x) >> 1;
  const int half = threadIdx.x & 1;
  if (t >= count) return;  // both lanes of a pair
  const uint32_t *p = (const uint32_t *)(pk + (size_t)t * P<LV>::PK);
  uint32_t a[25];
  shake256_absorb_pair<P<LV>::PK>(a, half, [&](int pos) { return p[pos / 4 + half]; });
  uint32_t *o = (uint32_t *)(out + (size_t)t * out_stride);
#pragma unroll
  for (int w = 0; w < P<LV>::TRB / 8; w++) o[2 * w + half] = a[w];
}

// the squeezed stream of one mask polynomial
template <int LV, class E>
__device__ __forceinline__ void dev_expand_mask_coop(const uint8_t *rhop, uint32_t nonce, const E &k, uint8_t *out) {
  constexpr int WPB = RATE256 / 4, NWORD = N * P<LV>::ZBITS / 32, NBLK = (NWORD + WPB - 1) / WPB;
  const uint32_t *rw = (const uint32_t *)rhop;
  uint32_t *o = (uint32_t *)out;
  uint32_t a[E::NR];
#pragma unroll
  for (int y = 0; y < E::NR; y++) {
    const int w = k.word(y);
    a[y] = w < 8 ? rw[k.half_word(y)] : 0u;
    if (w == 8 && !k.h) a[y] = (nonce & 0xFFFFu) | (0x1Fu << 16);
    if (w == RATE256 / 8 - 1 && k.h) a[y] = 0x80u << 24;
  }
#pragma unroll 1
  for (int blk = 0; blk < NBLK; blk++) {
    keccak_f_coop(a, k);
#pragma unroll
    for (int y = 0; y < E::NA; y++)
      if (k.own && k.word(y) < RATE256 / 8 && blk * WPB + k.half_word(y) < NWORD)
        o[blk * WPB + k.half_word(y)] = a[y];
  }
}

// as expand_mask_k
template <int LV, class E>
__global__ void __launch_bounds__(64) expand_mask_coop_k(Ws ws, const uint32_t *active, uint32_t count) {
  constexpr uint32_t ML = Lv<LV>::L;
  DIL_COOP_TASK(E)
  const uint32_t task = active[t / ML], i = t % ML;
  dev_expand_mask_coop<LV>(ws.rhop + (size_t)task * 64, ws.kappa[task] + i, k,
                           ws.y + ((size_t)task * ML + i) * P<LV>::YB);
}

// ---- KeyGen's seeds and the expansions of few keys, a wavefront per stream ----
// ExpandA of one polynomial: few of them leave a lane's five permutations (46 us
// one after another) alone on the chip.  The candidates of a block are tested on
// 56 lanes and placed by a ballot.  2,048 / 4,096 / 8,192 polynomials take 20 / 28 /
// 46 us this way, 59 each on lanes; beside the hash chains of Sign and Verify, which
// it delays above 4,096 (273 level-3 tasks of up to 4 KB, 8,190 polynomials: Verify
// 178 -> 183 us; 100 of 32 bytes, 3,000: 127 -> 98), the line lies there.
constexpr uint32_t EXPAND_BESIDE = 4096, EXPAND_ALONE = 8192;
struct ExpandLds {
  uint32_t kl[KECCAK_LDS], blk[RATE128 / 4 + 1];
  __align__(4) uint8_t poly[4 * N];
};
// rho(i): word i of the seed; out: A_POLY bytes, or 256 words (not PACKED)
template <bool PACKED, class R>
__device__ __forceinline__ void dev_expand_a_wave(R rho, uint32_t ij, uint8_t *out, const WaveKeccak &k,
                                                  ExpandLds &lds) {
  constexpr int POLY = PACKED ? A_POLY : 4 * N;
  uint32_t a[2];
#pragma unroll
  for (int y = 0; y < 2; y++) {
    const int w = k.word(y);
    a[y] = w < 4 ? rho(k.half_word(y)) : w == 4 && !k.h ? ij | 0x1Fu << 16 : 0u;
    if (w == RATE128 / 8 - 1 && k.h) a[y] ^= 0x80u << 24;
  }
  const bool cand = k.l < EA_CAND;
  const int wi = cand ? (3 * k.l) >> 2 : 0;
  const uint32_t sh = cand ? 8u * (uint32_t)((3 * k.l) & 3) : 0u;
  for (int ctr = 0; ctr < N;) {
    keccak_f_coop(a, k);
    if (k.own) {
      lds.blk[k.half_word(0)] = a[0];
      if (k.row == 0 && k.word(1) < RATE128 / 8) lds.blk[k.half_word(1)] = a[1];
    }
    wave_sync();
    const uint32_t v = __builtin_amdgcn_alignbit(lds.blk[wi + 1], lds.blk[wi], sh) & 0x7FFFFFu;
    const bool ok = cand && v < (uint32_t)Q;
    const uint64_t m = __ballot(ok);
    const int pos =
        ctr + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    if (ok && pos < N) {
      if constexpr (PACKED) {
        lds.poly[3 * pos] = (uint8_t)v;
        lds.poly[3 * pos + 1] = (uint8_t)(v >> 8);
        lds.poly[3 * pos + 2] = (uint8_t)(v >> 16);
      } else {
        ((uint32_t *)lds.poly)[pos] = v;
      }
    }
    ctr += (int)__popcll(m);
    wave_sync();
  }
#pragma unroll
  for (int q = 0; q < POLY / 256; q++) ((uint32_t *)out)[64 * q + k.l] = ((const uint32_t *)lds.poly)[64 * q + k.l];
}
// as expand_a_k
template <int LV>
__global__ void __launch_bounds__(64) expand_a_wave_k(const uint8_t *rho_src, size_t rho_stride, const uint32_t *key_idx,
                                                      uint8_t *A, uint32_t count) {
  constexpr uint32_t KL = Lv<LV>::K * Lv<LV>::L;
  __shared__ __align__(16) ExpandLds lds;
  const uint32_t task = blockIdx.x / KL, ij = blockIdx.x % KL;
  if (task >= count) return;
  const WaveKeccak k(lds.kl, threadIdx.x);
  const size_t key = key_idx ? key_idx[task] : task;
  const uint32_t *rho = (const uint32_t *)(rho_src + key * rho_stride);
  dev_expand_a_wave<true>([&](int i) { return rho[i]; }, ij % Lv<LV>::L | ij / Lv<LV>::L << 8,
                    A + (size_t)blockIdx.x * A_POLY, k, lds);
}
// as expand_a_seed_k
__global__ void __launch_bounds__(64) expand_a_seed_wave_k(const uint8_t *seeds, int32_t *out, uint32_t count) {
  __shared__ __align__(16) ExpandLds lds;
  if (blockIdx.x >= count) return;
  const WaveKeccak k(lds.kl, threadIdx.x);
  const uint8_t *sd = seeds + 34 * (size_t)blockIdx.x;
  dev_expand_a_wave<false>([&](int i) { return (uint32_t)load_le_bytes(sd + 4 * i, 4); },
                           (uint32_t)sd[32] | ((uint32_t)sd[33] << 8), (uint8_t *)(out + (size_t)blockIdx.x * N), k, lds);
}
// as kg_expand_k, ExpandS's streams after ExpandA's
template <int LV>
__global__ void __launch_bounds__(64) kg_expand_wave_k(const uint8_t *pk, Ws ws, uint32_t count) {
  constexpr uint32_t K = Lv<LV>::K, L = Lv<LV>::L, KL = K * L;
  __shared__ __align__(16) ExpandLds lds;
  const WaveKeccak k(lds.kl, threadIdx.x);
  if (blockIdx.x < count * KL) {
    const uint32_t task = blockIdx.x / KL, ij = blockIdx.x % KL;
    const uint32_t *rho = (const uint32_t *)(pk + (size_t)task * P<LV>::PK);
    dev_expand_a_wave<true>([&](int i) { return rho[i]; }, ij % L | ij / L << 8,
                      ws.A + (size_t)blockIdx.x * A_POLY, k, lds);
    return;
  }
  const uint32_t st = blockIdx.x - count * KL;
  if (st >= count * (K + L)) return;
  const uint32_t *rw = (const uint32_t *)(ws.rhop + (size_t)(st / (K + L)) * 64);
  uint32_t *o = (uint32_t *)(ws.s12 + (size_t)st * S_POLY);
  uint32_t a[2];
#pragma unroll
  for (int y = 0; y < 2; y++) {
    const int w = k.word(y);
    a[y] = w < 8 ? rw[k.half_word(y)] : w == 8 && !k.h ? st % (K + L) | 0x1Fu << 16 : 0u;
    if (w == RATE256 / 8 - 1 && k.h) a[y] = 0x80u << 24;
  }
  int got = 0;
  for (int blk = 0; blk < S_BLOCKS && (blk < 2 || got < N); blk++) {
    keccak_f_coop(a, k);
    const bool mine = k.own && k.word(0) < RATE256 / 8;
    if (mine) o[blk * (RATE256 / 4) + k.half_word(0)] = a[0];
    int c = mine ? (int)__popc(s_accepted<Lv<LV>::ETA>(a[0])) : 0;  // at most 8 a lane
#pragma unroll
    for (int bit = 0; bit < 4; bit++) got += (int)__popcll(__ballot((c >> bit) & 1)) << bit;
  }
}
// as kg_seed_k
template <int LV, class E>
__global__ void __launch_bounds__(64) kg_seed_coop_k(const uint8_t *seeds, uint8_t *pk, uint8_t *sk, Ws ws,
                                                     uint32_t count) {
  DIL_COOP_TASK(E)
  const uint8_t *sd = seeds + 32 * (size_t)t;
  uint32_t a[E::NR];
#pragma unroll
  for (int y = 0; y < E::NR; y++) {
    const int w = k.word(y);
    a[y] = w < 4 ? (uint32_t)load_le_bytes(sd + 4 * k.half_word(y), 4) : 0u;
    if (w == 4 && !k.h)
      a[y] = Lv<LV>::MLDSA ? (uint32_t)Lv<LV>::K | (uint32_t)Lv<LV>::L << 8 | 0x1Fu << 16 : 0x1Fu;
    if (w == RATE256 / 8 - 1 && k.h) a[y] = 0x80u << 24;
  }
  keccak_f_coop(a, k);
  uint32_t *pkw = (uint32_t *)(pk + (size_t)t * P<LV>::PK), *skw = (uint32_t *)(sk + (size_t)t * P<LV>::SK);
  uint32_t *rw = (uint32_t *)(ws.rhop + (size_t)t * 64);
#pragma unroll
  for (int y = 0; y < E::NA; y++) {
    const int i = k.half_word(y);
    if (!k.own || i >= 32) continue;
    if (i < 8) {
      pkw[i] = a[y];
      skw[i] = a[y];
    } else if (i < 24) {
      rw[i - 8] = a[y];
    } else {
      skw[i - 16] = a[y];  // K at sk bytes 32..63
    }
  }
}
#undef DIL_COOP_TASK

}  // namespace dil
