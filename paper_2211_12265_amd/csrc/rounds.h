// Sign in rounds (Alg. 2 loop), one launch per stage and round, with no host
// in the loop.
//
// A group of tasks goes through a fixed number of rounds.  In a round every
// unsigned task gets the same number of consecutive nonces (round_nonces in
// batch_sched.h), and four kernels run over
// all candidates: ExpandMask and the challenge (a lane, a lane pair, a 16-lane
// row or a wavefront per sponge, by their number), w = A y (one wavefront per
// candidate) and the checks (one wavefront per task going through its
// candidates in order, or a workgroup per task when m is large).  The checks stop at a task's first passing nonce, so
// the signature is the sequential algorithm's; tasks without one are appended
// to the next round's list and counted, and the next kernels read the count on
// the device.  Tasks still unsigned after the last round (about one in 10^2
// calls reaches that) are finished by the persistent kernel of persist.h,
// started at the next nonce (Resume).
//
// Against the persistent kernel, every stage gets the registers, the LDS and
// the wavefronts it wants: the loop kernel holds two wavefronts per SIMD for
// all stages and parks half of them while challenges are hashed.  Whole Sign
// call, loop kernel / rounds: 10,000 tasks at level 2 1465 / 1199 us, at level 5
// (32 to 4096-byte messages) 2844 / 2031 us; 2,503 hedged ML-DSA-65 1328 / 911
// us; 613 tasks on resident level-2 keys 834 / 460 us, one on a level-3 key
// 271 / 126 us.  With the kernels as they are now the rounds take 1043-1104, 1865-1889,
// 834-874, 337-412 and 83-97 us (the ranges are of different cards).
#pragma once
#include <algorithm>

#include "keccak_row.h"
#include "persist.h"

namespace dil {

constexpr int ROUNDS_MAX = 8;
constexpr int ROUND_WORDS = 16;  // counter words of a group: [r] unfinished tasks at the start of round r > 0,
                                 // [ROUNDS_MAX + 1] work queue of the finishing kernel
static_assert(ROUNDS_MAX + 2 <= ROUND_WORDS, "a group's counters");

// One group: tasks [first, first + n) of the call; cap = round_candidates(n).
struct Group {
  uint32_t first, n, cap;
  uint32_t *cnt;      // [ROUND_WORDS], zeroed before the first round
  uint32_t *list[2];  // unsigned tasks of odd / even rounds, [n] each (round 0 takes all, in order)
  uint8_t *y;         // [cap][L][YB]
  int32_t *w;         // [cap][K][256], register order
  uint8_t *w1;        // [cap][K * W1B]
  uint8_t *ct;        // [cap][CT_STRIDE]
  int8_t *c;          // [cap][256]
};

// task of entry e of round r's list
__device__ __forceinline__ uint32_t round_task(const Group &gr, int r, uint32_t e) {
  return r == 0 ? gr.first + e : gr.list[r & 1][e];
}

// ExpandMask streams: a round of many has one lane each; as long as the chip
// would hold at most one wavefront per SIMD, a stream gets a lane pair, and
// with still fewer a 16-lane row or a whole wavefront (two per SIMD).  A stream
// is five permutations one after another and a lone wavefront's permutation
// takes 9.2 us on one lane, 6.8 us on a pair, 3.1 us on a row and 2.5 us over
// the wavefront; beyond these counts the wider forms would queue for the SIMDs.
constexpr uint32_t PAIR_STATES = 32768;
inline uint32_t mask_blocks(uint64_t streams, bool exact) {
  // 256-lane workgroups that the form of at most `streams` streams needs (exact: of that many)
  auto need = [](uint64_t n) -> uint64_t {
    return n <= WAVE_STATES ? (n + 3) / 4 : n <= ROW_STATES ? (n + 15) / 16 : n <= PAIR_STATES ? (n + 127) / 128 : (n + 255) / 256;
  };
  uint64_t b = need(streams);
  if (!exact) {
    if (streams > WAVE_STATES) b = b > need(WAVE_STATES) ? b : need(WAVE_STATES);
    if (streams > ROW_STATES) b = b > need(ROW_STATES) ? b : need(ROW_STATES);
    if (streams > PAIR_STATES) b = b > need(PAIR_STATES) ? b : need(PAIR_STATES);
  }
  return (uint32_t)b;
}

// the squeezed stream of one candidate polynomial on a lane pair
template <int LV>
__device__ __forceinline__ void dev_expand_mask_pair(const uint8_t *rhop, uint32_t nonce, int half, uint8_t *out) {
  constexpr int WPB = RATE256 / 4, NWORD = N * P<LV>::ZBITS / 32, NBLK = (NWORD + WPB - 1) / WPB;
  const uint32_t *rw = (const uint32_t *)rhop;
  uint32_t *o = (uint32_t *)out + half;
  uint32_t a[25];
#pragma unroll
  for (int i = 0; i < 25; i++) a[i] = i < 8 ? rw[2 * i + half] : 0u;
  if (!half) a[8] = (nonce & 0xFFFFu) | (0x1Fu << 16);
  else a[RATE256 / 8 - 1] = 0x80u << 24;
#pragma unroll
  for (int blk = 0; blk < NBLK; blk++) {
    keccak_f_pair(a, half);
#pragma unroll
    for (int i = 0; i < WPB / 2; i++)
      if (blk * WPB + 2 * i < NWORD) o[blk * WPB + 2 * i] = a[i];
  }
}
template <int LV>
__global__ void __launch_bounds__(256) rd_mask_k(Ws ws, Group gr, int r) {
  constexpr uint32_t L = Lv<LV>::L;
  __shared__ uint32_t kl[4][KECCAK_LDS];
  __builtin_amdgcn_s_setprio(2);
  const RoundState st = round_state(gr.cnt, gr.n, r);
  const uint32_t total = st.n * st.m * L;
  const uint32_t lanes = total <= WAVE_STATES ? 64 : total <= ROW_STATES ? 16 : total <= PAIR_STATES ? 2 : 1;
  const uint32_t id = (blockIdx.x * 256 + threadIdx.x) / lanes;
  if (id >= total) return;
  const uint32_t s = id / L, i = id - s * L, e = s / st.m;
  const uint8_t *rhop = ws.rhop + (size_t)round_task(gr, r, e) * 64;
  const uint32_t kappa = (st.first + (s - e * st.m)) * L;
  uint8_t *out = gr.y + (size_t)id * P<LV>::YB;
  if (lanes == 1) {
    dev_expand_mask<LV>(rhop, kappa, (int)i, out);
  } else if (lanes == 2) {
    dev_expand_mask_pair<LV>(rhop, kappa + i, threadIdx.x & 1, out);
  } else if (lanes == 16) {
    dev_expand_mask_coop<LV>(rhop, kappa + i, RowKeccak(kl[threadIdx.x >> 6], threadIdx.x & 63), out);
  } else {
    dev_expand_mask_coop<LV>(rhop, kappa + i, WaveKeccak(kl[threadIdx.x >> 6], threadIdx.x & 63), out);
  }
}

// w = INTT(A NTT(y)) and its packed high bits: one wavefront per candidate.
// Four candidates per workgroup, so that candidates of one task mostly share
// a CU and read its A-hat from the vector cache once.
template <int LV>
struct RoundWLds {
  int32_t hat[Lv<LV>::L * HAT_POLY];
  int32_t tr[4 * NTT_LDS_GROUP];
  uint32_t w1buf[Lv<LV>::K * P<LV>::W1B / 4 + 1];
};
template <int LV>
__global__ void __launch_bounds__(256) rd_w_k(Ws ws, Group gr, int r) {
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L;
  __shared__ __align__(16) RoundWLds<LV> lds[4];
  const RoundState st = round_state(gr.cnt, gr.n, r);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, t = lane & 15;
  const uint32_t s = blockIdx.x * 4 + wave;
  if (s >= st.n * st.m) return;
  const uint32_t task = round_task(gr, r, s / st.m);
  const Tw ftw = ntt_lane_tw(t), itw = intt_lane_tw(t);
  RoundWLds<LV> &l = lds[wave];
  dev_compute_w<LV, true, true, 4, false>(gr.y + (size_t)s * L * P<LV>::YB, ws.A + kix(ws, task) * K * L * A_POLY, gr.w + (size_t)s * K * N,
                    gr.w1 + (size_t)s * K * P<LV>::W1B, l.hat, l.tr + (lane >> 4) * NTT_LDS_GROUP, l.w1buf, ftw, itw,
                    lane);
}

// ctilde = H(mu || w1), c = SampleInBall(ctilde): two lanes per candidate, a
// 16-lane row as long as that takes at most two wavefronts per SIMD, or a
// wavefront (eight permutations in series: 65 us on pairs, 43 on rows, 26 on
// wavefronts)
inline uint32_t chal_blocks(uint32_t cand) {
  const uint32_t waves = std::min(cand, WAVE_STATES), rows = (std::min(cand, ROW_ALONE) + 3) / 4,
                 pairs = (cand + 31) / 32;
  return std::max(waves, std::max(rows, pairs));
}
template <int LV>
__global__ void __launch_bounds__(64) rd_chal_k(Ws ws, Group gr, int r) {
  __shared__ __align__(16) int8_t cl[32][C_ROW];
  __shared__ uint32_t bb[32][RATE256 / 4];
  __shared__ uint32_t kl[KECCAK_LDS];
  __builtin_amdgcn_s_setprio(3);
  const RoundState st = round_state(gr.cnt, gr.n, r);
  const uint32_t total = st.n * st.m;
  const int lane = threadIdx.x, per = total <= WAVE_STATES ? 1 : total <= ROW_ALONE ? 4 : 32;
  const int p = per == 1 ? 0 : per == 4 ? lane >> 4 : lane >> 1;
  const uint32_t s = blockIdx.x * per + p;
  if (s >= total) return;  // a whole pair, row or wavefront
  const uint32_t task = round_task(gr, r, s / st.m);
  const uint8_t *mu = ws.muw1 + (size_t)task * muw1_stride<LV>();
  const uint8_t *w1 = gr.w1 + (size_t)s * Lv<LV>::K * P<LV>::W1B;
  uint32_t *ct = (uint32_t *)(gr.ct + (size_t)s * CT_STRIDE);
  int8_t *c = gr.c + (size_t)s * N;
  if (per == 1) {
    const WaveKeccak k(kl, lane);
    dev_challenge_coop<LV>(mu, w1, k, ct, cl[0], bb[0]);
    store_c_coop(cl[0], c, k);
  } else if (per == 4) {
    const RowKeccak k(kl, lane);
    dev_challenge_coop<LV>(mu, w1, k, ct, cl[p], bb[p]);
    store_c_coop(cl[p], c, k);
  } else {
    dev_challenge_pair<LV>(mu, w1, lane & 1, ct, cl[p], bb[p]);
    wave_sync();
    const uint32_t *cw = (const uint32_t *)cl[p];
    for (int v = lane & 1; v < N / 16; v += 2)
      ((int4 *)c)[v] = make_int4(cw[4 * v], cw[4 * v + 1], cw[4 * v + 2], cw[4 * v + 3]);
  }
}

// The checks.  Up to ROUND_SEQ nonces per task, each wavefront takes a task and
// evaluates its candidates in order, so that none after the first passing one
// is looked at; with more, the four wavefronts of a workgroup share a task.
// Three wavefronts per SIMD (168 registers, of which l = 7 spills 9): with two, which
// need no spills, levels 5 and 87 take 0-1% longer from 2,500 tasks on and 1-2% less
// below 300.
constexpr uint32_t ROUND_SEQ = 6;
template <int LV>
__global__ void __launch_bounds__(256, 3) rd_check_k(Ws ws, Group gr, uint8_t *sig, int r, uint32_t *stats) {
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L;
  __shared__ __align__(16) CheckLds<LV> lds[4];
  __shared__ uint32_t seq;
  __shared__ int okw[4];
  const RoundState st = round_state(gr.cnt, gr.n, r);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (blockIdx.x == 0 && threadIdx.x == 0)
    atomicAdd((unsigned long long *)&stats[2], (unsigned long long)st.n * st.m);
  const bool shared = st.m > ROUND_SEQ;  // uniform over the launch
  const uint32_t e = shared ? blockIdx.x : blockIdx.x * 4 + wave;
  if ((shared ? e : blockIdx.x * 4) >= st.n) return;
  if (threadIdx.x == 0) seq = 0;
  __syncthreads();
  const bool live = e < st.n;
  const uint32_t task = live ? round_task(gr, r, e) : 0;
  uint32_t win = SCHED_NONE;
  for (uint32_t k0 = 0; k0 < st.m && win == SCHED_NONE; k0 += shared ? 4 : 1) {
    const uint32_t k = shared ? k0 + wave : k0;
    bool ok = false;
    if (live && k < st.m) {
      const size_t s = (size_t)e * st.m + k;
      ok = dev_check<LV>(gr.c + s * N, (const uint32_t *)(gr.ct + s * CT_STRIDE), gr.y + s * L * P<LV>::YB,
                         gr.w + s * K * N, ws.sec + kix(ws, task) * sec_bytes<LV>(), lds[wave], lane);
    }
    if (shared) {
      if (lane == 0) okw[wave] = ok;
      __syncthreads();
      for (int v = 3; v >= 0; v--)
        if (okw[v]) win = k0 + v;
      __syncthreads();
    } else if (ok) {
      win = k;
    }
  }
  if (live) {
    if (win != SCHED_NONE) {
      if (!shared || (win & 3) == (uint32_t)wave) {
        l2g_bytes(lds[wave].sigbuf, P<LV>::SIG, sig + (size_t)task * P<LV>::SIG, lane, 64);
        if (lane == 0) atomicAdd(&seq, st.first + win + 1);
      }
    } else if (lane == 0 && (!shared || wave == 0)) {
      gr.list[(r + 1) & 1][atomicAdd(&gr.cnt[r + 1], 1u)] = task;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && seq) atomicAdd((unsigned long long *)&stats[6], (unsigned long long)seq);
}

// ---- one candidate by one workgroup of l wavefronts ----
// With few candidates every stage is one chain on a nearly idle chip, and what
// counts is the length of the chains and of the way between them: mask
// polynomial i on wavefront i, w on eight 16-lane groups of two wavefronts (one
// pass of each transform instead of two at l > 4), the challenge on the first one,
// with the packed HighBits(w) still in LDS.
template <int LV>
struct CandLds {
  uint32_t kl[Lv<LV>::L][KECCAK_LDS];
  union {
    struct {
      int32_t hat[Lv<LV>::L * HAT_POLY];
      int32_t tr[8 * NTT_LDS_GROUP];
      uint32_t w1buf[Lv<LV>::K * P<LV>::W1B / 4 + 1];
    };
    CheckLds<LV> ck;
  };
  __align__(16) int8_t c[N];
  uint32_t ct[P<LV>::CT / 4];
  int ok;
};
// y to y_out, w to w_out, ctilde and c to lds; k: the wavefront's engine on its
// lds.kl.  All wavefronts call; only the first may read ct and c without a barrier.
template <int LV>
__device__ __forceinline__ void dev_candidate(const uint8_t *rhop, uint32_t kappa, const uint8_t *A, const uint8_t *mu,
                                              uint8_t *y_out, int32_t *w_out, const WaveKeccak &k, CandLds<LV> &lds) {
  static_assert(Lv<LV>::L >= 2, "two wavefronts for w");
  const int tid = threadIdx.x, wave = tid >> 6, t = tid & 15;
  dev_expand_mask_coop<LV>(rhop, kappa + wave, k, y_out + wave * P<LV>::YB);
  __syncthreads();
  if (wave < 2) {
    const Tw ftw = ntt_lane_tw(t), itw = intt_lane_tw(t);
    dev_compute_w<LV, true, true, 8>(y_out, A, w_out, nullptr, lds.hat, lds.tr + (tid >> 4) * NTT_LDS_GROUP, lds.w1buf,
                                     ftw, itw, tid);
  } else {  // its two barriers
    __syncthreads();
    __syncthreads();
  }
  if (wave == 0) dev_challenge_coop<LV>(mu, (const uint8_t *)lds.w1buf, k, lds.ct, lds.c, nullptr);
}

// Masks, w and challenges of a round of at most CAND_TASKS tasks, whose
// candidates (64 per task) then have a workgroup each: 49 us for one task of
// level 3, 63 us in three launches (and their gaps).
constexpr uint32_t CAND_TASKS = 8;
template <int LV>
__global__ void __launch_bounds__(64 * Lv<LV>::L) rd_cand_k(Ws ws, Group gr, int r) {
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L;
  __shared__ __align__(16) CandLds<LV> lds;
  const RoundState st = round_state(gr.cnt, gr.n, r);
  const uint32_t s = blockIdx.x;
  if (s >= st.n * st.m) return;
  const uint32_t e = s / st.m, task = round_task(gr, r, e);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const WaveKeccak k(lds.kl[wave], lane);
  dev_candidate<LV>(ws.rhop + (size_t)task * 64, (st.first + (s - e * st.m)) * L, ws.A + kix(ws, task) * K * L * A_POLY,
                    ws.muw1 + (size_t)task * muw1_stride<LV>(), gr.y + (size_t)s * L * P<LV>::YB,
                    gr.w + (size_t)s * K * N, k, lds);
  if (wave != 0) return;
  wave_sync();
  if (lane < P<LV>::CT / 4) ((uint32_t *)(gr.ct + (size_t)s * CT_STRIDE))[lane] = lds.ct[lane];
  store_c_coop(lds.c, gr.c + (size_t)s * N, k);
}

// The staged form's loop for the tasks of a list that are few enough for a
// workgroup each: up to `most` nonces (at most FEW_TRIES), in order, until one passes.  A round in
// four launches and a wait of the host took 83 us with a few tasks left, a nonce
// here takes 50 (level 3; 1,000 tasks 3000 -> 2170 us).  Two wavefronts per SIMD:
// with three dev_check spills at every level (2,230 us; level 5 2,000 against 1,850);
// with two, 10 registers at l = 7 and none elsewhere.
constexpr uint32_t FEW_TRIES = 64, FEW_STREAMS = WAVE_STATES;
template <int LV>
__global__ void __launch_bounds__(64 * Lv<LV>::L, 2) sg_few_k(Ws ws, uint8_t *sig, const uint32_t *active, uint32_t nactive,
                                                            uint32_t *next_active, uint32_t most) {
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L;
  __shared__ __align__(16) CandLds<LV> lds;
  if (blockIdx.x >= nactive) return;
  const uint32_t task = active[blockIdx.x];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const WaveKeccak k(lds.kl[wave], lane);
  uint8_t *y = ws.y + (size_t)task * L * P<LV>::YB;
  int32_t *w = ws.w + (size_t)task * K * N;
  const uint32_t kappa = ws.kappa[task];
  uint32_t tries = 0;
  bool done;
  do {
    dev_candidate<LV>(ws.rhop + (size_t)task * 64, kappa + tries * L, ws.A + kix(ws, task) * K * L * A_POLY,
                      ws.muw1 + (size_t)task * muw1_stride<LV>(), y, w, k, lds);
    tries++;
    if (wave == 0) {
      wave_sync();
      const bool ok = dev_check<LV>(lds.c, lds.ct, y, w, ws.sec + kix(ws, task) * sec_bytes<LV>(), lds.ck, lane);
      if (ok) l2g_bytes(lds.ck.sigbuf, P<LV>::SIG, sig + (size_t)task * P<LV>::SIG, lane, 64);
      if (lane == 0) lds.ok = ok;
    }
    __syncthreads();
    done = lds.ok;
  } while (!done && tries < most);
  if (threadIdx.x == 0) {
    atomicAdd(&ws.counters[1], tries);
    if (!done) {
      ws.kappa[task] = kappa + tries * L;
      next_active[atomicAdd(&ws.counters[0], 1u)] = task;
    }
  }
}

}  // namespace dil
