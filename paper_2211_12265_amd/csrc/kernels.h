// Batched Dilithium kernels for gfx950 (Alg. 1-3), one-launch-per-stage form.
//
// Thread mappings:
//   sponge kernels      one lane per SHAKE stream (256-thread blocks)
//   polynomial kernels  one wavefront per task, four 16-lane groups each
//                       working on its own polynomial (64-thread blocks)
// All intermediates live in a per-task workspace in HBM (see Ws).
#pragma once
#include "common.h"
#include "ntt.h"
#include "poly.h"
#include "sponge.h"
#include "keccak_pair.h"
#include "toeplitz.h"

namespace dil {

// Per-task workspace of the staged kernels.  Rows are 256-byte aligned; the
// hash inputs mu || packed w1 are stored contiguously, in the order the hash
// consumes them, so the challenge hash reads one row.
struct Ws {
  uint8_t *muw1;     // [cap][MUW1 rounded to 256]
  uint8_t *rhop;     // [cap][64]   rho' (KeyGen: expanded secret seed; Sign: mask seed)
  uint8_t *ctilde;   // [cap][CT_STRIDE]
  int8_t *cpoly;     // [cap][256]  challenge c, dense
  uint8_t *A;        // [cap][K][L][A_POLY]  A-hat, 24 bits per coefficient (load_a)
  uint8_t *s12;      // KeyGen: the streams of s1, s2, [cap][L+K][S_POLY]
  int8_t *sec;       // [cap][sec_bytes] Sign: s1, s2, t0 as int8 tiles (toeplitz.h)
  uint8_t *y;        // [cap][L][YB]  mask, as squeezed
  int32_t *w;        // [cap][K][256]  w = A y as dev_compute_w stores it
  uint32_t *kappa;   // [cap]
  int32_t *flag;     // [cap]
  uint32_t *active0, *active1;  // [cap] task lists
  uint32_t *counters;           // [8]: next active count, error flags, attempts
  // Resident key tables: when kmap is set, A, sec (and t1s, tr) are
  // indexed by key row kmap[task] instead of by task.
  const uint32_t *kmap;
  const int8_t *t1s;    // [keys][TILE_BYTES] t1 as an int8 tile (verify), or null
  const uint8_t *tr;    // [keys][TRB] tr = H(pk) (verify), or null
};

constexpr int CT_STRIDE = 64;  // workspace row of a ctilde (the longest, ML-DSA-87's)

// bytes hashed before the message for mu: tr (round 3), tr || 0x00 || 0x00
// (ML-DSA, empty context) or tr alone before a formatted message (ML-DSA's
// internal form)
template <int LV, bool INTERNAL>
constexpr int mu_prefix_bytes() {
  static_assert(!INTERNAL || Lv<LV>::MLDSA, "formatted messages exist at the ML-DSA levels only");
  return !Lv<LV>::MLDSA ? 32 : INTERNAL ? 64 : 66;
}

// row of the per-key arrays used by task `task`
__device__ __forceinline__ size_t kix(const Ws &ws, uint32_t task) { return ws.kmap ? ws.kmap[task] : task; }

template <int LV>
__host__ __device__ __forceinline__ size_t muw1_stride() {
  return ((size_t)P<LV>::MUW1 + 255) & ~(size_t)255;
}

// zero two word arrays with one workgroup (used instead of hipMemsetAsync so that the
// launch sequence can be captured into a hipGraph)
__global__ void zero_words_k(uint32_t *a, int na, uint32_t *b, int nb) {
  for (int i = threadIdx.x; i < na; i += blockDim.x) a[i] = 0;
  if (b)
    for (int i = threadIdx.x; i < nb; i += blockDim.x) b[i] = 0;
}

// The first launch of a call: zeroes two word arrays (workgroup 0) and, in
// key-table calls (key_idx set), copies key_idx into the workspace with every
// index outside the table replaced by row 0 and the error word set, so no later
// kernel reads past the table; the host reports the error at its next check.
__global__ void __launch_bounds__(256) begin_k(uint32_t *a, int na, uint32_t *b, int nb, const uint32_t *key_idx,
                                               uint32_t nkeys, uint32_t *out, uint32_t count, uint32_t *err) {
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < na; i += 256) a[i] = 0;
    for (int i = threadIdx.x; i < nb; i += 256) b[i] = 0;
  }
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (!key_idx || i >= count) return;
  uint32_t k = key_idx[i];
  if (k >= nkeys) {
    k = 0;
    *err = 1u;
  }
  out[i] = k;
}

// ------------------------------------------------------------------------
// KeyGen (Alg. 1)
// ------------------------------------------------------------------------
// (rho, rho', K) = H(zeta): rho -> pk and sk, K -> sk, rho' -> workspace.
// ML-DSA hashes xi || k || l (one byte each) instead of the bare seed.
template <int LV>
__global__ void __launch_bounds__(256) kg_seed_k(const uint8_t *seeds, uint8_t *pk, uint8_t *sk, Ws ws,
                                                 uint32_t count) {
  uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count) return;
  uint32_t s[50];
  const uint8_t *sd = seeds + 32 * (size_t)t;
  shake_absorb<RATE256>(s, Lv<LV>::MLDSA ? 34 : 32, [&](uint64_t pos) -> uint64_t {
    return pos < 32 ? load_le_bytes(sd + pos, 8) : (uint64_t)Lv<LV>::K | ((uint64_t)Lv<LV>::L << 8);
  });
  uint64_t *pkw = (uint64_t *)(pk + (size_t)t * P<LV>::PK);
  uint64_t *skw = (uint64_t *)(sk + (size_t)t * P<LV>::SK);
  uint64_t *rw = (uint64_t *)(ws.rhop + (size_t)t * 64);
#pragma unroll
  for (int w = 0; w < 16; w++) {
    uint64_t v = (uint64_t)s[2 * w] | ((uint64_t)s[2 * w + 1] << 32);
    if (w < 4) {
      pkw[w] = v;
      skw[w] = v;
    } else if (w < 12) {
      rw[w - 4] = v;
    } else {
      skw[w - 8] = v;  // K at sk bytes 32..63
    }
  }
}

// ExpandA (Sec. 2.3 sampling; Alg. 4's rejection sampler): 3 bytes -> 23-bit
// candidate, kept if < q, in stream order, until 256 are kept.  One lane per
// SHAKE128 stream; only 1 in 1,024 candidates is rejected, so 95% of the blocks
// of 56 are kept whole and the lane stores them itself, 16 bytes at a time at
// its position, with no exchange between lanes.  The other lanes' blocks (3.4
// of 64 per squeeze) are compacted by the wavefront: staged in LDS, tested on
// 56 lanes at once, a ballot gives each accepted candidate its position.
// Bound by the issue of the Keccak instructions (21.6 k of the wavefront's 23 k);
// testing every block on 56 lanes took 5.3 k more.  2^20 polynomials 710 -> 630 us,
// 300,000 beside nothing 281 -> 218 us.
// out0 is lane 0's polynomial, lane l's the l-th after it.  rows: EA_ROWS * EA_ROW
// words of LDS for this wavefront.  Lanes with valid = false run the
// permutations but store nothing.
constexpr int EA_CAND = RATE128 / 3;      // 56 candidates per block
constexpr int EA_ROW = RATE128 / 4 + 1;   // 43 words: the last candidate's second word is read too
constexpr int EA_ROWS = 16;               // blocks compacted per pass
constexpr int EA_WG = 64;                 // one wavefront per workgroup
constexpr int EA_FULL = N / EA_CAND;      // 4 blocks are needed whole, at least
constexpr int EA_LAST = N - EA_FULL * EA_CAND;  // candidates of the next one when nothing was rejected
static_assert(EA_CAND % 4 == 0 && EA_LAST % 16 == 0, "stored in fours, and in 16 bytes when packed");

// 16 bytes at a polynomial's next free place, which a rejection leaves at any byte
template <int ALIGN>
struct __attribute__((packed, aligned(ALIGN))) EaQuad {
  uint32_t v[4];
};
template <int ALIGN>
struct __attribute__((packed, aligned(ALIGN))) EaPair {
  uint32_t v[2];
};

// PACKED: polynomials of A_POLY bytes, 24 bits per coefficient as squeezed (bit 23
// is not part of it), else 256 words each.
template <bool PACKED>
__device__ __forceinline__ void expand_a_squeeze_wave(uint32_t s[50], uint8_t *out0, uint32_t *rows, int lane,
                                                      bool valid) {
  constexpr int POLY = PACKED ? A_POLY : 4 * N, CB = PACKED ? 3 : 4;  // bytes per polynomial, per coefficient
  int ctr = valid ? 0 : N;
  uint8_t *out = out0 + (size_t)lane * POLY;
  // lane l < 56 tests candidate l of a staged block: bytes 3l .. 3l + 2, inside words wi and wi + 1
  const bool cand = lane < EA_CAND;
  const int wi = cand ? (3 * lane) >> 2 : 0;
  const uint32_t sh = cand ? 8u * (uint32_t)((3 * lane) & 3) : 0u;
#pragma unroll 1
  for (int blk = 0;; blk++) {
    // the lane's own candidates, four per three words
    uint32_t tv[EA_CAND], top = 0, top_last = 0;
#pragma unroll
    for (int k = 0; k < EA_CAND / 4; k++) {
      tv[4 * k] = s[3 * k] & 0x7FFFFFu;
      tv[4 * k + 1] = __builtin_amdgcn_alignbit(s[3 * k + 1], s[3 * k], 24) & 0x7FFFFFu;
      tv[4 * k + 2] = __builtin_amdgcn_alignbit(s[3 * k + 2], s[3 * k + 1], 16) & 0x7FFFFFu;
      tv[4 * k + 3] = (s[3 * k + 2] >> 8) & 0x7FFFFFu;
      top = max(top, max(max(tv[4 * k], tv[4 * k + 1]), max(tv[4 * k + 2], tv[4 * k + 3])));
      if (4 * k + 4 == EA_LAST) top_last = top;
    }
    const bool whole = blk < EA_FULL && top < (uint32_t)Q && ctr < N;
    const bool tail = blk == EA_FULL && top_last < (uint32_t)Q && ctr == N - EA_LAST;
    if (whole || tail) {
      uint8_t *o = out + CB * ctr;
      if constexpr (PACKED) {
#pragma unroll
        for (int k = 0; k < RATE128 / 16; k++)
          if (16 * k < 3 * EA_LAST || whole)
            ((EaQuad<1> *)o)[k] = EaQuad<1>{{s[4 * k], s[4 * k + 1], s[4 * k + 2], s[4 * k + 3]}};
        if (whole) *(EaPair<1> *)(o + RATE128 / 16 * 16) = EaPair<1>{{s[RATE128 / 4 - 2], s[RATE128 / 4 - 1]}};
      } else {
#pragma unroll
        for (int k = 0; k < EA_CAND / 4; k++)
          if (4 * k < EA_LAST || whole)
            ((EaQuad<4> *)o)[k] = EaQuad<4>{{tv[4 * k], tv[4 * k + 1], tv[4 * k + 2], tv[4 * k + 3]}};
      }
      ctr += whole ? EA_CAND : EA_LAST;
    }
    // blocks with a rejection (or, at the end, after one)
    uint64_t left = __ballot(!(whole || tail) && ctr < N);
    while (left) {
      const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(left >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)left, 0u));
      if (((left >> lane) & 1) && rank < EA_ROWS) {
#pragma unroll
        for (int w = 0; w < RATE128 / 4; w++) rows[rank * EA_ROW + w] = s[w];
      }
      wave_sync();
#pragma unroll 1
      for (int r = 0; r < EA_ROWS && left; r++) {
        const int L = __builtin_ctzll(left);
        left &= left - 1;
        const uint32_t *row = rows + r * EA_ROW;
        const uint32_t v = __builtin_amdgcn_alignbit(row[wi + 1], row[wi], sh) & 0x7FFFFFu;
        const int cL = __builtin_amdgcn_readlane(ctr, L);
        const bool ok = cand && v < (uint32_t)Q;
        const uint64_t m = __ballot(ok);
        const int pos =
            cL + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (ok && pos < N) {
          uint8_t *o = out0 + (size_t)L * POLY + CB * pos;
          if constexpr (PACKED) {
            o[0] = (uint8_t)v;
            o[1] = (uint8_t)(v >> 8);
            o[2] = (uint8_t)(v >> 16);
          } else {
            *(uint32_t *)o = v;
          }
        }
        if (lane == L) ctr = min(N, cL + (int)__popcll(m));
      }
      wave_sync();
    }
    if (blk >= EA_FULL && __ballot(ctr < N) == 0) break;
    keccak_f(s);
  }
}

// ExpandA: one lane per (task, i, j); rho read from rows of `rho_src` (pk or sk).
// WG: lanes per workgroup; rows: EA_ROWS * EA_ROW words per wavefront.
template <int LV, int WG>
__device__ __forceinline__ void dev_expand_a(uint32_t block, const uint8_t *rho_src, size_t rho_stride,
                                             const uint32_t *key_idx, uint8_t *A, uint32_t count, uint32_t *rows) {
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L;
  const int lane = threadIdx.x & 63;
  const uint64_t st = (uint64_t)block * WG + threadIdx.x;
  const bool valid = st < (uint64_t)count * K * L;
  const uint64_t sl = valid ? st : 0;
  uint32_t task = (uint32_t)(sl / (K * L));
  int ij = (int)(sl % (K * L));
  int i = ij / L, j = ij % L;
  size_t key = key_idx ? key_idx[task] : task;
  const uint64_t *rho = (const uint64_t *)(rho_src + key * rho_stride);
  uint32_t s[50];
  absorb_seed34(s, [&](int pos) { return rho[pos >> 3]; }, (uint32_t)j | ((uint32_t)i << 8));
  expand_a_squeeze_wave<true>(s, A + (size_t)(st - lane) * A_POLY, rows + (threadIdx.x >> 6) * EA_ROWS * EA_ROW, lane,
                              valid);
}
template <int LV, int WG = EA_WG>
__global__ void __launch_bounds__(WG) expand_a_k(const uint8_t *rho_src, size_t rho_stride, const uint32_t *key_idx,
                                                  uint8_t *A, uint32_t count) {
  __shared__ uint32_t rows[WG / 64 * EA_ROWS * EA_ROW];
  dev_expand_a<LV, WG>(blockIdx.x, rho_src, rho_stride, key_idx, A, count, rows);
}

// KeyGen's ExpandA and ExpandS, which need nothing of each other, in one launch:
// the first nblk_a workgroups are ExpandA's, the others have one lane per (task,
// r < L + K) of ExpandS and fill the SIMDs as those of ExpandA run out.
template <int LV>
__global__ void __launch_bounds__(EA_WG) kg_expand_k(const uint8_t *pk, Ws ws, uint32_t count, uint32_t nblk_a) {
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L;
  __shared__ uint32_t rows[EA_ROWS * EA_ROW];
  if (blockIdx.x < nblk_a) {
    dev_expand_a<LV, EA_WG>(blockIdx.x, pk, P<LV>::PK, nullptr, ws.A, count, rows);
    return;
  }
  const uint64_t st = (uint64_t)(blockIdx.x - nblk_a) * EA_WG + threadIdx.x;
  if (st >= (uint64_t)count * (K + L)) return;
  uint32_t s[50];
  absorb_seed66(s, ws.rhop + st / (K + L) * 64, (uint32_t)(st % (K + L)));
  expand_s_squeeze<Lv<LV>::ETA>(s, ws.s12 + st * S_POLY);
}

// LDS layout shared by the per-task polynomial kernels
template <int LV>
struct PolyLds {
  int32_t tr[4 * NTT_LDS_GROUP];              // transposes, one region per group
  int32_t hat[(Lv<LV>::L > Lv<LV>::K ? Lv<LV>::L : Lv<LV>::K) * HAT_POLY];  // NTT-domain vector (hat_idx)
  uint32_t buf[(P<LV>::SK + 64) / 4 + 2];     // byte staging (packed rows), + pad words
};

// consecutive-layout values of the lane (16t .. 16t+15) from its strided values
template <bool PAD = true>
__device__ __forceinline__ void to_consecutive(const int32_t x[16], uint32_t v[16], int32_t *tr, int t) {
  int32_t y[16];
#pragma unroll
  for (int r = 0; r < 16; r++) y[r] = x[r];
  transpose_s2c<PAD>(y, tr, t);
#pragma unroll
  for (int r = 0; r < 16; r++) v[r] = (uint32_t)y[r];
}

// The polynomial of an ExpandS stream by a 16-lane group: eta - s of its 256
// coefficients as bytes in buf (LDS).  A lane takes 32 nibbles of the first 256
// bytes, its place comes from the lanes before it; what is missing after them
// (one polynomial of 500) from 16 bytes at a time.
template <int ETA>
__device__ __forceinline__ void dev_collect_s(const uint8_t *src, uint8_t *buf, int t) {
  auto scan = [&](int c, int &total) {  // sum over the group's lanes before this one
    int s = c;
    s += (int)row_shr<1>((uint32_t)s);
    s += (int)row_shr<2>((uint32_t)s);
    s += (int)row_shr<4>((uint32_t)s);
    s += (int)row_shr<8>((uint32_t)s);
    total = __shfl(s, 15, 16);
    return s - c;
  };
  auto put = [&](uint32_t w, uint32_t ok, int nibbles, int pos) {
    uint32_t v[2] = {w & 0x0F0F0F0Fu, (w >> 4) & 0x0F0F0F0Fu};
    if constexpr (ETA == 2)  // v mod 5 for v < 15; 13 v < 2^8
      for (int q = 0; q < 2; q++) v[q] -= 5u * ((13u * v[q] >> 6) & 0x03030303u);
#pragma unroll
    for (int b = 0; b < nibbles; b++) {
      const bool keep = (ok >> (4 * b)) & 1;
      if (keep && pos < N) buf[pos] = (uint8_t)(v[b & 1] >> (8 * (b >> 1)));
      pos += keep;
    }
    return pos;
  };
  const uint4 q = ((const uint4 *)src)[t];
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
  uint32_t ok[4];
  int c = 0, got;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    ok[i] = s_accepted<ETA>(w[i]);
    c += __popc(ok[i]);
  }
  int pos = scan(c, got);
#pragma unroll
  for (int i = 0; i < 4; i++) pos = put(w[i], ok[i], 8, pos);
  for (int o = 16 * 16; o < S_POLY && got < N; o += 16) {
    const uint32_t b = src[o + t], k = s_accepted<ETA>(b) & 0x11u;
    int more;
    put(b, k, 2, got + scan(__popc(k), more));
    got += more;
  }
  wave_sync();
}
// ... its packed coefficients' words (consecutive layout) and its coefficients (strided layout)
template <int ETA>
__device__ __forceinline__ void load_s(const uint8_t *buf, uint32_t v[16], int32_t x[16], int t) {
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const uint32_t w = ((const uint32_t *)buf)[4 * t + q];
#pragma unroll
    for (int b = 0; b < 4; b++) v[4 * q + b] = (w >> (8 * b)) & 0xFFu;
  }
#pragma unroll
  for (int r = 0; r < 16; r++) x[r] = ETA - (int32_t)buf[t + 16 * r];
  wave_sync();
}

// KeyGen main: t = INTT(A * NTT(s1)) + s2, Power2Round, pack pk's t1 and sk's
// s1, s2, t0.  One wavefront per key; LDS holds only what the kernel writes of pk
// and sk, which decides how many wavefronts a CU takes.
template <int LV>
__global__ void __launch_bounds__(64) kg_main_k(Ws ws, uint8_t *pk, uint8_t *sk, uint32_t count) {
  using PP = P<LV>;
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L, ETA = Lv<LV>::ETA;
  constexpr int SKW = (PP::SK - PP::OFF_S1) / 4, PKW = (PP::PK - 32) / 4;
  __shared__ int32_t trl[4 * NTT_LDS_GROUP];
  __shared__ int32_t hat[L * HAT_POLY];
  __shared__ uint32_t skbuf[SKW], pkbuf[PKW];
  const uint32_t task = blockIdx.x;
  if (task >= count) return;
  int lane = threadIdx.x, g = lane >> 4, t = lane & 15;
  int32_t *tr = trl + g * NTT_LDS_GROUP;
  uint8_t *skb = (uint8_t *)skbuf;
  uint8_t *pkb = (uint8_t *)pkbuf;
  const uint8_t *S = ws.s12 + (size_t)task * (K + L) * S_POLY;
  const Tw ftw = ntt_lane_tw(t), itw = intt_lane_tw(t);
  // s1: NTT into LDS, and pack eta - s into sk
  for (int j = g; j < L; j += 4) {
    int32_t x[16];
    uint32_t v[16];
    dev_collect_s<ETA>(S + j * S_POLY, (uint8_t *)tr, t);
    load_s<ETA>((const uint8_t *)tr, v, x, t);
    pack16_to_lds<PP::EBITS>(v, skb + j * PP::EB, t);
    ntt16(x, ftw, tr, t);
#pragma unroll
    for (int r = 0; r < 16; r++) hat[hat_idx(j, t, r)] = x[r];
  }
  wave_sync();
  for (int i = g; i < K; i += 4) {
    const uint8_t *Ai = ws.A + ((size_t)task * K + i) * L * A_POLY;
    int64_t acc[16];
#pragma unroll
    for (int r = 0; r < 16; r++) acc[r] = 0;
    for (int j = 0; j < L; j++) {
      int32_t a[16];
      load_a(a, Ai + j * A_POLY, t);
#pragma unroll
      for (int r = 0; r < 16; r++) acc[r] += (int64_t)a[r] * hat[hat_idx(j, t, r)];
    }
    int32_t x[16];
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = mont_reduce(acc[r]);
    intt16(x, itw, tr, t);
    int32_t s2[16];
    uint32_t v[16];
    dev_collect_s<ETA>(S + (L + i) * S_POLY, (uint8_t *)tr, t);
    load_s<ETA>((const uint8_t *)tr, v, s2, t);
    pack16_to_lds<PP::EBITS>(v, skb + (PP::OFF_S2 - PP::OFF_S1) + i * PP::EB, t);
    int32_t t1[16], t0[16];
#pragma unroll
    for (int r = 0; r < 16; r++) {
      int32_t tv = canon(x[r]) + s2[r];            // in [-eta, q + eta)
      tv += (tv >> 31) & Q;
      tv -= Q;
      tv += (tv >> 31) & Q;                        // canonical
      power2round(tv, t1[r], t0[r]);
      t0[r] = (1 << (D - 1)) - t0[r];
    }
    to_consecutive(t1, v, tr, t);
    pack16_to_lds<10>(v, pkb + i * PP::T1B, t);
    to_consecutive(t0, v, tr, t);
    pack16_to_lds<13>(v, skb + (PP::OFF_T0 - PP::OFF_S1) + i * PP::T0B, t);
  }
  wave_sync();
  // copy the packed regions out (pk[32..PK), sk[OFF_S1..SK)); rho, K, tr are written elsewhere
  uint32_t *pkg = (uint32_t *)(pk + (size_t)task * PP::PK + 32);
  for (int w = lane; w < PKW; w += 64) pkg[w] = pkbuf[w];
  uint32_t *skg = (uint32_t *)(sk + (size_t)task * PP::SK + PP::OFF_S1);
  for (int w = lane; w < SKW; w += 64) skg[w] = skbuf[w];
}

// ------------------------------------------------------------------------
// Sign (Alg. 2), staged
// ------------------------------------------------------------------------
// mu and the mask seed of task t on a lane pair (keccak_pair.h; both lanes
// call); initialises kappa and the active list.
//   round 3: mu = H(tr || M); rho' = H(K || mu), or the task's 64 rnd bytes
//            themselves (randomized signing) when rnd is not null;
//   ML-DSA:  mu = H(tr || 0x00 || 0x00 || M); rho'' = H(K || rnd || mu) with
//            the task's 32 rnd bytes, or 32 zero bytes when rnd is null;
//            with INTERNAL the messages are formatted messages M' (a context
//            string or the pre-hash form, built by the caller) and mu =
//            H(tr || M').
// rnd rows are 4-byte aligned.
template <int LV, bool INTERNAL = false>
__device__ __forceinline__ void dev_prep_pair(uint32_t t, int half, const uint8_t *sk, const uint32_t *key_idx,
                                              const uint8_t *msg, const uint64_t *msg_off, const uint8_t *rnd,
                                              const Ws &ws, uint32_t *err) {
  size_t key = key_idx ? key_idx[t] : t;
  const uint8_t *skr = sk + key * P<LV>::SK;
  uint64_t o0 = msg_off[t], o1 = msg_off[t + 1];
  uint64_t mlen = 0;
  if (o1 >= o0) mlen = o1 - o0;
  else if (!half) atomicOr(err, 1u);  // decreasing msg_off: message treated as empty
  constexpr int TW = P<LV>::TRB / 4;
  uint32_t a[25];
  uint32_t trw[TW];
  const uint32_t *skw = (const uint32_t *)(skr + 64);  // tr inside the 8-byte aligned sk row
#pragma unroll
  for (int i = 0; i < TW; i++) trw[i] = skw[i];
  absorb_prefix_msg<mu_prefix_bytes<LV, INTERNAL>()>(a, half, trw, msg + o0, mlen);
  uint32_t mu[8];  // this lane's halves of mu's eight 8-byte words
  uint32_t *muw = (uint32_t *)(ws.muw1 + (size_t)t * muw1_stride<LV>());
#pragma unroll
  for (int i = 0; i < 8; i++) {
    mu[i] = a[i];
    muw[2 * i + half] = a[i];
  }
  uint32_t *rp = (uint32_t *)(ws.rhop + (size_t)t * 64);
  if constexpr (Lv<LV>::MLDSA) {
    // rho'' = H(K || rnd || mu): 128 bytes, one block
    const uint32_t *Kw = (const uint32_t *)(skr + 32);
    const uint32_t *rw = rnd ? (const uint32_t *)(rnd + (size_t)t * 32) : nullptr;
#pragma unroll
    for (int i = 0; i < 25; i++)
      a[i] = i < 4 ? Kw[2 * i + half] : i < 8 ? (rw ? rw[2 * (i - 4) + half] : 0u) : i < 16 ? mu[i - 8] : 0u;
    a[16] ^= half ? 0x80u << 24 : 0x1Fu;
    keccak_f_pair(a, half);
#pragma unroll
    for (int i = 0; i < 8; i++) rp[2 * i + half] = a[i];
  } else if (rnd) {
    const uint32_t *rw = (const uint32_t *)(rnd + (size_t)t * 64);
#pragma unroll
    for (int i = 0; i < 8; i++) rp[2 * i + half] = rw[2 * i + half];
  } else {
    // rho' = H(K || mu): 96 bytes, one block
    const uint32_t *Kw = (const uint32_t *)(skr + 32);
#pragma unroll
    for (int i = 0; i < 25; i++) a[i] = i < 4 ? Kw[2 * i + half] : i < 12 ? mu[i - 4] : 0u;
    if (!half) a[12] ^= 0x1Fu;
    else a[RATE256 / 8 - 1] ^= 0x80u << 24;
    keccak_f_pair(a, half);
#pragma unroll
    for (int i = 0; i < 8; i++) rp[2 * i + half] = a[i];
  }
  if (!half) {
    ws.kappa[t] = 0;
    ws.active0[t] = t;
  }
}

// s1, s2 and t0 unpacked from sk into the int8 tiles of toeplitz.h, one
// wavefront per key row: lane chunk id = 64 k + lane holds coefficients
// 16 (id & 15) .. + 15 of tile row id >> 4, so that a wavefront's 16-byte
// stores are contiguous.  Bound by memory: 2.5 / 4 / 4.9 KB read and 4 / 8 / 8
// KB written per key at levels 2 / 3 / 5 (the NTT-domain int32 form it
// replaces wrote 12 / 17 / 23 KB and ran 12 / 17 / 23 transforms).
template <int LV>
__global__ void __launch_bounds__(64) sg_secret_k(const uint8_t *sk, const uint32_t *key_idx, Ws ws, uint32_t count) {
  using PP = P<LV>;
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L, ETA = Lv<LV>::ETA;
  constexpr int NW = (PP::SK - PP::OFF_S1) / 4;
  __shared__ uint32_t buf[NW + 2];
  const uint32_t task = blockIdx.x;
  if (task >= count) return;
  const int lane = threadIdx.x;
  size_t key = key_idx ? key_idx[task] : task;
  // stage sk bytes OFF_S1..SK into LDS (sk rows are 8-byte aligned)
  g2l_words<NW>((const uint32_t *)(sk + key * PP::SK + PP::OFF_S1), buf, lane);
  if (lane < 2) buf[NW + lane] = 0;
  wave_sync();
  v4i *out = (v4i *)(ws.sec + (size_t)task * sec_bytes<LV>());
  const int part = (lane >> 4) & 3, c0 = 16 * (lane & 15);
#pragma unroll 1
  for (int k = 0; k < 4 * sec_tiles<LV>(); k++) {  // the wavefront's four rows: the parts of polynomial k
    uint32_t v[4] = {0, 0, 0, 0};
    if (part < 2) {
      if (k < (part ? K : L)) {
        const uint32_t *src = buf + (part ? L + k : k) * (PP::EB / 4);
#pragma unroll
        for (int r = 0; r < 16; r++)
          v[r >> 2] |= (uint32_t)((ETA - (int32_t)field<PP::EBITS>(src, c0 + r)) & 0xFF) << (8 * (r & 3));
      }
    } else if (k < K) {
      const uint32_t *src = buf + ((L + K) * PP::EB + k * PP::T0B) / 4;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int32_t t0 = (1 << (D - 1)) - (int32_t)field<13>(src, c0 + r), hi = (t0 + 32) >> 6;
        v[r >> 2] |= (uint32_t)((part == 2 ? t0 - 64 * hi : hi) & 0xFF) << (8 * (r & 3));
      }
    }
    out[64 * k + lane] = v4i{(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
  }
}

// ---- Sign iteration building blocks, shared by the staged kernels and the
// ---- persistent kernel (same arithmetic in both execution forms)

// ExpandMask stream i of iteration kappa (one lane)
template <int LV>
__device__ __forceinline__ void dev_expand_mask(const uint8_t *rhop, uint32_t kappa, int i, uint8_t *y_out) {
  uint32_t s[50];
  absorb_seed66(s, rhop, (kappa + (uint32_t)i) & 0xFFFFu);
  expand_mask_squeeze<P<LV>::ZBITS>(s, y_out);
}

// w = INTT(A-hat * NTT(y)) for one task by one wavefront: w as the checks take it
// (pack_low; each lane's 16 strided coefficients contiguous: word 16 t + r of a
// polynomial is coefficient t + 16 r) to w_out, HighBits(w) packed into w1_out (4-byte aligned, K * W1B bytes).
// hat: L * HAT_POLY words of LDS; tr: this group's transpose region; w1buf: LDS
// staging; ftw / itw: forward / inverse twiddles.
// EARLY: the group's first A-hat polynomial (row g, column 0) is requested
// before the NTT of y, and each next one before the current one is multiplied.
// The fences of the NTT's LDS transposes keep the compiler from hoisting these
// loads by itself, which leaves each load's latency exposed; requesting them
// early costs 12 registers per lane, which only the l = 4 loop kernels have.
// NG: 16-lane groups that share the work; with more than a wavefront's four, all
// wavefronts of the workgroup meet at two barriers, and the packed HighBits(w)
// stay in w1buf.
// TOGETHER: as in load_mask.
template <int LV, bool PAD = true, bool EARLY = false, int NG = 4, bool TOGETHER = true, class TW>
__device__ __forceinline__ void dev_compute_w(const uint8_t *y, const uint8_t *A, int32_t *w_out, uint8_t *w1_out,
                                              int32_t *hat, int32_t *tr, uint32_t *w1buf, const TW &ftw,
                                              const TW &itw, int lane) {
  using PP = P<LV>;
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L;
  int g = lane >> 4, t = lane & 15;
  APart an;
  if constexpr (EARLY) {
    if (g < K) an.load(A + (size_t)g * L * A_POLY, t);
  }
  for (int j = g; j < L; j += NG) {
    int32_t x[16];
    load_mask<PP::ZBITS, Lv<LV>::GAMMA1, TOGETHER>(x, y + j * PP::YB, t);
    ntt16<TW, PAD>(x, ftw, tr, t);
#pragma unroll
    for (int r = 0; r < 16; r++) hat[hat_idx(j, t, r)] = x[r];
  }
  if constexpr (NG > 4) __syncthreads();
  else wave_sync();
  for (int i = g; i < K; i += NG) {
    const uint8_t *Ai = A + (size_t)i * L * A_POLY;
    int64_t acc[16];
#pragma unroll
    for (int r = 0; r < 16; r++) acc[r] = 0;
    if constexpr (EARLY) {
      for (int j = 0; j < L; j++) {
        int32_t a[16];
        an.get(a);
        if (j + 1 < L) an.load(Ai + (j + 1) * A_POLY, t);
        else if (i + NG < K) an.load(A + (size_t)(i + NG) * L * A_POLY, t);
#pragma unroll
        for (int r = 0; r < 16; r++) acc[r] += (int64_t)a[r] * hat[hat_idx(j, t, r)];
      }
    } else {
      for (int j = 0; j < L; j++) {
        int32_t a[16];
        load_a(a, Ai + j * A_POLY, t);
#pragma unroll
        for (int r = 0; r < 16; r++) acc[r] += (int64_t)a[r] * hat[hat_idx(j, t, r)];
      }
    }
    int32_t x[16];
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = mont_reduce(acc[r]);
    intt16<TW, PAD>(x, itw, tr, t);
    int32_t w1[16];
#pragma unroll
    for (int r = 0; r < 16; r++) {
      int32_t r0;
      decompose<LV>(canon(x[r]), w1[r], r0);
      x[r] = pack_low(w1[r], r0);
    }
    store_slots(x, w_out + i * N, t);
    uint32_t v[16];
    to_consecutive<PAD>(w1, v, tr, t);
    pack16_to_lds<PP::W1BITS>(v, (uint8_t *)w1buf + i * PP::W1B, t);
  }
  if constexpr (NG > 4) {
    __syncthreads();
  } else {
    wave_sync();
    uint32_t *dst = (uint32_t *)w1_out;
    for (int w = lane; w < K * PP::W1B / 4; w += 64) dst[w] = w1buf[w];
  }
}

// SampleInBall on the lane's SHAKE256(ctilde) stream, into a per-lane 256-byte
// LDS array; positions are drawn with rejection against the loop index.
template <int TAU>
__device__ __forceinline__ void sample_in_ball(uint32_t s[50], int8_t *c, uint8_t *blockbuf) {
  // s holds the first squeezed block
  uint32_t *bw = (uint32_t *)blockbuf;
#pragma unroll
  for (int w = 0; w < RATE256 / 4; w++) bw[w] = s[w];
  uint64_t signs = (uint64_t)s[0] | ((uint64_t)s[1] << 32);
  uint32_t *cw = (uint32_t *)c;
#pragma unroll
  for (int w = 0; w < N / 4; w++) cw[w] = 0;
  int pos = 8;
  for (int i = N - TAU; i < N; i++) {
    int b;
    for (;;) {
      if (pos == RATE256) {
        keccak_f(s);
#pragma unroll
        for (int w = 0; w < RATE256 / 4; w++) bw[w] = s[w];
        pos = 0;
      }
      b = blockbuf[pos++];
      if (b <= i) break;
    }
    c[i] = c[b];
    c[b] = (int8_t)(1 - 2 * (int)(signs & 1));
    signs >>= 1;
  }
}

// ctilde = H(mu || w1) of CT bytes (mu and packed w1 8-byte aligned);
// c = SampleInBall(ctilde), seeded by all of ctilde (one lane)
template <int LV>
__device__ __forceinline__ void dev_challenge(const uint8_t *mu, const uint8_t *w1, uint32_t *ctilde_out, int8_t *c,
                                              uint8_t *blockbuf) {
  constexpr int CW = P<LV>::CT / 4;
  uint32_t s[50];
  shake_absorb<RATE256>(s, P<LV>::MUW1, [&](uint64_t pos) {
    return pos < 64 ? *(const uint64_t *)(mu + pos) : *(const uint64_t *)(w1 + (pos - 64));
  });
  uint32_t ct[CW];
#pragma unroll
  for (int i = 0; i < CW; i++) {
    ct[i] = s[i];
    ctilde_out[i] = s[i];
  }
  keccak_zero(s);
#pragma unroll
  for (int i = 0; i < CW; i++) s[i] = ct[i];
  s[CW] = 0x1Fu;
  s[2 * (RATE256 / 8 - 1) + 1] ^= 0x80u << 24;
  keccak_f(s);
  sample_in_ball<Lv<LV>::TAU>(s, c, blockbuf);
}

template <int LV>
struct CheckLds {
  uint32_t ct[TOEP_WORDS];               // shifted copies of the challenge (toeplitz.h)
  uint32_t sigbuf[P<LV>::SIG / 4 + 2];   // packed signature; holds f while the copies are built
  uint16_t hmask[Lv<LV>::K][16];
  int rowcnt[Lv<LV>::K];
};

// The rejection checks of Alg. 2 for one candidate (one wavefront):
// z = y + c s1, r0 = LowBits(w - c s2), c t0 and the hint.  c is the dense
// challenge (int8, natural order, 4-byte aligned), sec the key's int8 tiles.
// Returns true (wave-uniform) if the candidate passes all four checks; the
// packed signature (ctilde, z, h) is then in lds.sigbuf.
//
// The products by c run on the matrix cores (toeplitz.h): 64 products per tile
// of four polynomials, exact, instead of one NTT and twelve INTTs of four
// polynomials each and no reductions mod q afterwards.  Group g evaluates
// polynomial 4 T + g of tile T; w comes as dev_compute_w stores it; a tile whose z or r0 norm fails ends the
// evaluation before its c t0, hints and packing (about 77% of the candidates
// at level 2).  z is packed by OR-ing each strided coefficient's bits into the
// signature: only passing tiles pay for it, and no transpose is needed.
// Measured against the transforms it replaces (10,000 tasks, whole Sign call,
// four-wavefront loop kernel): level 2 1470 to 1410 us, level 5 2799 to 2680 us;
// staged form, level 3, 1000 tasks: 6996 to 6725 us.
template <int LV>
__device__ __forceinline__ bool dev_check(const int8_t *c, const uint32_t *ctilde, const uint8_t *y, const int32_t *w,
                                          const int8_t *sec, CheckLds<LV> &lds, int lane) {
  using PP = P<LV>;
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L, BETA = Lv<LV>::BETA, OMEGA = Lv<LV>::OMEGA;
  constexpr int32_t G1 = Lv<LV>::GAMMA1, G2 = Lv<LV>::GAMMA2;
  static_assert(sizeof lds.sigbuf >= 129 * 4, "the build scratch lies in the signature buffer");
  const int g = lane >> 4, t = lane & 15;
  uint8_t *sb = (uint8_t *)lds.sigbuf;
  // the operands of the first tile are requested before the copies are built
  const uint32_t cw = ((const uint32_t *)c)[lane];
  v4i s[4];
  toep_load(s, sec, lane);
  int32_t yv[16], wv[16], ct0[16];
  static_assert(K >= 4 && L >= 4, "the first tile is full");
  load_mask<PP::ZBITS, G1>(yv, y + g * PP::YB, t);
  load_slots(wv, w + g * N, t);
  toep_build(cw, lds.ct, lds.sigbuf, lane);
  for (int q = lane; q < (int)(sizeof lds.sigbuf / 4); q += 64) lds.sigbuf[q] = 0;
  wave_sync();
#pragma unroll 1
  for (int T = 0; T < sec_tiles<LV>(); T++) {
    const int p = 4 * T + g;
    const bool hz = L % 4 == 0 || p < L, hr = K % 4 == 0 || p < K;  // every group has work in a full tile
    if (T > 0) {
      if (hz) load_mask<PP::ZBITS, G1>(yv, y + p * PP::YB, t);
      if (hr) load_slots(wv, w + p * N, t);
    }
    // |z| < gamma1 - beta, as an offset maximum, and |r0| < gamma2 - beta from the extremes of w - c s2
    uint32_t zm = 0;
    int32_t wmax = 0, wmin = 0;
    auto half = [&](auto I0c) {
      constexpr int I0 = decltype(I0c)::value;
      v4i acc[8];
      toep_mul<I0, 8>(acc, s, lds.ct, lane);
      if (hz) {
#pragma unroll
        for (int r = 0; r < 8; r++) {
          yv[I0 + r] += acc[r][0];
          zm = max(zm, (uint32_t)(yv[I0 + r] + (G1 - BETA - 1)));
        }
      }
      if (hr) {
#pragma unroll
        for (int r = 0; r < 8; r++) {
          wv[I0 + r] -= acc[r][1] * (1 << LOW_SHIFT);  // high bits of w, low part minus c s2
          wmax = max(wmax, wv[I0 + r]);
          wmin = min(wmin, wv[I0 + r]);
          ct0[I0 + r] = acc[r][2] + 64 * acc[r][3];
        }
      }
    };
    half(std::integral_constant<int, 0>{});
    __builtin_amdgcn_sched_barrier(0);  // or both halves' reads are hoisted and their registers held at once
    half(std::integral_constant<int, 8>{});
    if (wave_any(zm > 2u * (G1 - BETA - 1))) return false;
    if (wave_any(low_fails<G2, BETA>(wmax) || low_fails<G2, BETA>(wmin))) {
      if (!wave_any(low_beyond<G2, BETA>(wmax) || low_beyond<G2, BETA>(wmin))) return false;
      // a key row with s2 beyond eta (lowbits.h)
      bool fails = false;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        wv[r] = low_carry<G2, PP::M_HB>(wv[r]);
        fails |= low_fails<G2, BETA>(wv[r]);
      }
      if (wave_any(hr && fails)) return false;
    }
    if (T + 1 < sec_tiles<LV>()) toep_load(s, sec + (T + 1) * TILE_BYTES, lane);
    bool bad = false;
    if (hr) {
      int cnt = 0;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        bad |= (uint32_t)(ct0[r] + (G2 - 1)) > 2u * (G2 - 1);
        const bool h = hint_of<G2>(low_part(wv[r]) + ct0[r], low_high(wv[r]));
        const uint64_t m = __ballot(h);
        const uint32_t m16 = (uint32_t)(m >> (16 * g)) & 0xFFFFu;
        if (t == 0) lds.hmask[p][r] = (uint16_t)m16;
        cnt += __popc(m16);
      }
      if (t == 0) lds.rowcnt[p] = cnt;
    }
    if (wave_any(bad)) return false;
    if (hz) {
      // coefficient t + 16 r is the B-bit field at bit B t + 16 B r of row p, and 16 B r is a whole number of words
      constexpr int B = PP::ZBITS;
      uint32_t *zw = lds.sigbuf + (PP::OFF_Z + p * PP::ZB) / 4 + ((B * t) >> 5);
      const int sh = (B * t) & 31;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const uint64_t v = (uint64_t)(uint32_t)(G1 - yv[r]) << sh;
        atomicOr(zw + r * (B / 2), (uint32_t)v);
        if (sh + B > 32) atomicOr(zw + r * (B / 2) + 1, (uint32_t)(v >> 32));
      }
    }
  }
  wave_sync();
  int total = 0;
  for (int i = 0; i < K; i++) total += lds.rowcnt[i];
  if (total > OMEGA) return false;
  // accepted: ctilde and the hint bytes (the buffer is zeroed)
  if (lane < PP::CT / 4) lds.sigbuf[lane] = ctilde[lane];
  for (int i = g; i < K; i += 4) {
    int pre = 0;
    for (int i2 = 0; i2 < i; i2++) pre += lds.rowcnt[i2];
#pragma unroll
    for (int r = 0; r < 16; r++) {
      uint32_t m16 = lds.hmask[i][r];
      if ((m16 >> t) & 1u) sb[PP::OFF_H + pre + __popc(m16 & ((1u << t) - 1u))] = (uint8_t)(t + 16 * r);
      pre += __popc(m16);
    }
    if (t == 0) sb[PP::OFF_H + OMEGA + i] = (uint8_t)pre;
  }
  wave_sync();
  return true;
}

// ---- staged kernels ----
// ExpandMask: one lane per (active task, i < L)
template <int LV>
__global__ void __launch_bounds__(256) expand_mask_k(Ws ws, const uint32_t *active, uint32_t nactive) {
  constexpr int L = Lv<LV>::L;
  uint64_t st = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (st >= (uint64_t)nactive * L) return;
  uint32_t task = active[st / L];
  int i = (int)(st % L);
  dev_expand_mask<LV>(ws.rhop + (size_t)task * 64, ws.kappa[task], i, ws.y + ((size_t)task * L + i) * P<LV>::YB);
}

// w = INTT(A * NTT(y)); w1 = HighBits(w) packed after mu
template <int LV>
__global__ void __launch_bounds__(64) sg_w_k(Ws ws, const uint32_t *active, uint32_t nactive) {
  using PP = P<LV>;
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L;
  __shared__ PolyLds<LV> lds;
  if (blockIdx.x >= nactive) return;
  uint32_t task = active[blockIdx.x];
  int lane = threadIdx.x, t = lane & 15;
  const Tw ftw = ntt_lane_tw(t), itw = intt_lane_tw(t);
  dev_compute_w<LV>(ws.y + (size_t)task * L * P<LV>::YB, ws.A + kix(ws, task) * K * L * A_POLY, ws.w + (size_t)task * K * N,
                    ws.muw1 + (size_t)task * muw1_stride<LV>() + 64, lds.hat, lds.tr + (lane >> 4) * NTT_LDS_GROUP,
                    lds.buf, ftw, itw, lane);
  (void)PP::K;
}

// One lane's dense challenge in LDS: rows of C_ROW bytes (65 words), so that
// the lanes of a wavefront writing the same coefficient index hit 64
// different banks; copied out to a 16-byte aligned global row.
constexpr int C_ROW = N + 4;
__device__ __forceinline__ void store_c_row(const int8_t *c, int8_t *dst) {
  const uint32_t *cw = (const uint32_t *)c;
  int4 *d = (int4 *)dst;
#pragma unroll
  for (int w = 0; w < N / 16; w++) d[w] = make_int4(cw[4 * w], cw[4 * w + 1], cw[4 * w + 2], cw[4 * w + 3]);
}

// ctilde = H(mu || w1); c = SampleInBall(ctilde).  One lane per active task.
template <int LV>
__global__ void __launch_bounds__(64) sg_chal_k(Ws ws, const uint32_t *active, uint32_t nactive) {
  __shared__ int8_t cl[64][C_ROW];
  __shared__ uint32_t bb[64][RATE256 / 4];
  uint32_t a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= nactive) return;
  uint32_t task = active[a];
  int8_t *c = cl[threadIdx.x];
  const uint8_t *row = ws.muw1 + (size_t)task * muw1_stride<LV>();
  dev_challenge<LV>(row, row + 64, (uint32_t *)(ws.ctilde + (size_t)task * CT_STRIDE), c, (uint8_t *)bb[threadIdx.x]);
  store_c_row(c, ws.cpoly + (size_t)task * N);
}

// checks; accept -> signature row of the task, reject -> kappa += l and next round.
// Left alone, the compiler adds AGPRs for dev_check's accumulators (174 registers at
// level 2); in 126 / 128 / 144 nothing spills.
template <int LV>
__global__ void __launch_bounds__(64, Lv<LV>::K > 6 ? 2 : 3) sg_check_k(Ws ws, uint8_t *sig, const uint32_t *active, uint32_t nactive,
                                                 uint32_t *next_active) {
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L;
  __shared__ __align__(16) CheckLds<LV> lds;
  if (blockIdx.x >= nactive) return;
  uint32_t task = active[blockIdx.x];
  const int lane = threadIdx.x;
  bool ok = dev_check<LV>(ws.cpoly + (size_t)task * N, (const uint32_t *)(ws.ctilde + (size_t)task * CT_STRIDE),
                          ws.y + (size_t)task * L * P<LV>::YB, ws.w + (size_t)task * K * N,
                          ws.sec + kix(ws, task) * sec_bytes<LV>(), lds, lane);
  if (ok) {
    l2g_bytes(lds.sigbuf, P<LV>::SIG, sig + (size_t)task * P<LV>::SIG, lane, 64);
  } else if (lane == 0) {
    ws.kappa[task] += L;
    uint32_t slot = atomicAdd(&ws.counters[0], 1u);
    next_active[slot] = task;
  }
}

// ------------------------------------------------------------------------
// Verify (Alg. 3), staged
// ------------------------------------------------------------------------
// tr = H(pk) (unless resident) and mu = H(tr || M) (ML-DSA: H(tr || 0x00 ||
// 0x00 || M), or H(tr || M') of formatted messages with INTERNAL) of task t on a
// lane pair (keccak_pair.h; both lanes call)
template <int LV, bool INTERNAL = false>
__device__ __forceinline__ void dev_hash_pair(uint32_t t, int half, const uint8_t *pk, const uint32_t *key_idx,
                                              const uint8_t *msg, const uint64_t *msg_off, const Ws &ws,
                                              uint32_t *err) {
  using PP = P<LV>;
  size_t key = key_idx ? key_idx[t] : t;
  uint64_t o0 = msg_off[t], o1 = msg_off[t + 1];
  uint64_t mlen = 0;
  if (o1 >= o0) mlen = o1 - o0;
  else if (!half) atomicOr(err, 1u);  // decreasing msg_off: message treated as empty
  constexpr int TW = PP::TRB / 4;
  uint32_t a[25];
  uint32_t trw[TW];
  if (ws.tr) {
    const uint32_t *tg = (const uint32_t *)(ws.tr + key * PP::TRB);
#pragma unroll
    for (int i = 0; i < TW; i++) trw[i] = tg[i];
  } else {
    const uint32_t *pkr = (const uint32_t *)(pk + key * PP::PK);
    shake256_absorb_pair<PP::PK>(a, half, [&](int pos) { return pkr[pos / 4 + half]; });
    // both lanes need all of tr: the partner's halves come over the DPP swap
#pragma unroll
    for (int i = 0; i < TW / 2; i++) {
      const uint32_t other = pair_swap(a[i]);
      trw[2 * i] = half ? other : a[i];
      trw[2 * i + 1] = half ? a[i] : other;
    }
  }
  absorb_prefix_msg<mu_prefix_bytes<LV, INTERNAL>()>(a, half, trw, msg + o0, mlen);
  uint32_t *muw = (uint32_t *)(ws.muw1 + (size_t)t * muw1_stride<LV>());
#pragma unroll
  for (int i = 0; i < 8; i++) muw[2 * i + half] = a[i];
}

// c = SampleInBall(ctilde), one lane per task
template <int LV>
__global__ void __launch_bounds__(64) vf_prep_k(const uint8_t *sig, Ws ws, uint32_t count) {
  using PP = P<LV>;
  __shared__ int8_t cl[64][C_ROW];
  __shared__ uint32_t bb[64][RATE256 / 4];
  uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count) return;
  const uint8_t *sg = sig + (size_t)t * PP::SIG;
  uint32_t s[50];
  // all CT bytes of ctilde
  keccak_zero(s);
#pragma unroll
  for (int w = 0; w < PP::CT / 8; w++) {
    uint64_t v = load_le_bytes(sg + 8 * w, 8);
    s[2 * w] = (uint32_t)v;
    s[2 * w + 1] = (uint32_t)(v >> 32);
  }
  s[PP::CT / 4] = 0x1Fu;
  s[2 * (RATE256 / 8 - 1) + 1] ^= 0x80u << 24;
  keccak_f(s);
  int8_t *c = cl[threadIdx.x];
  sample_in_ball<Lv<LV>::TAU>(s, c, (uint8_t *)bb[threadIdx.x]);
  store_c_row(c, ws.cpoly + (size_t)t * N);
}

// Strict decoding of the OMEGA + K hint bytes hb (LDS) into hm[K][8] (LDS, bit
// masks) by one wavefront, byte j on lane j mod 64.  Returns whether this
// lane's bytes break a rule: counts non-decreasing and at most OMEGA, indices
// strictly increasing within a polynomial, unused bytes zero.
template <int LV>
__device__ __forceinline__ bool dev_decode_hints(const uint8_t *hb, uint32_t *hm, int lane) {
  constexpr int K = Lv<LV>::K, OMEGA = Lv<LV>::OMEGA;
  static_assert(8 * K <= 64 && OMEGA <= 128, "one mask word and two hint bytes per lane at most");
  if (lane < 8 * K) hm[lane] = 0;
  wave_sync();
  bool bad = false;
  int cnt[K], prev = 0;
#pragma unroll
  for (int i = 0; i < K; i++) {
    cnt[i] = hb[OMEGA + i];
    bad |= cnt[i] < prev || cnt[i] > OMEGA;
    prev = cnt[i];
  }
#pragma unroll
  for (int q = 0; q < 2; q++) {
    const int j = lane + 64 * q;
    if (j < OMEGA) {
      const uint32_t v = hb[j];
      int i = 0, start = 0;  // polynomial of byte j and its first byte
#pragma unroll
      for (int p = 0; p < K; p++)
        if (j >= cnt[p]) {
          i = p + 1;
          start = cnt[p];
        }
      if (i >= K) bad |= v != 0;
      else {
        if (j > start) bad |= v <= hb[j - 1];
        atomicOr(&hm[8 * i + (v >> 5)], 1u << (v & 31));
      }
    }
  }
  wave_sync();
  return bad;
}

// LDS of the main part of Verify.  The signature's bytes are dead once z and the
// hints are unpacked; the copies of the challenge and the packed w1' rows take
// their place.
template <int LV>
struct VfLds {
  static constexpr int SIGW = P<LV>::SIG / 4 + 3, W1W = Lv<LV>::K * P<LV>::W1B / 4 + 1, TW = TOEP_WORDS + 132;
  __align__(16) int32_t trl[4 * NTT_LDS_GROUP];
  int32_t zh[Lv<LV>::L * HAT_POLY];
  __align__(16) uint32_t region[SIGW > TW + W1W ? SIGW : TW + W1W];
  uint32_t hm[8 * Lv<LV>::K];
};
// w1' = UseHint(h, INTT(A NTT(z)) - c t1 2^d), packed after mu; z norm check and
// hint decoding.  One wavefront per task; cw: the lane's word of the dense
// challenge.  c t1 comes from the matrix cores (toeplitz.h) after the INTT, which
// leaves two NTT passes of four polynomials per four rows: NTT(c) and
// NTT(t1 2^d) ran as two more (level 3, 10,000 tasks: 128 us, now 106).
template <int LV>
__device__ __forceinline__ void dev_vf_main(uint32_t task, uint32_t cw, VfLds<LV> &lds, const uint8_t *pk,
                                            const uint32_t *key_idx, const uint8_t *sig, const Ws &ws) {
  using PP = P<LV>;
  constexpr int K = Lv<LV>::K, L = Lv<LV>::L, BETA = Lv<LV>::BETA;
  constexpr int32_t G1 = Lv<LV>::GAMMA1;
  int32_t *const trl = lds.trl, *const zh = lds.zh;
  uint32_t *const region = lds.region, *const hm = lds.hm;
  uint32_t *const sigw = region, *const ct = region, *const w1b = region + VfLds<LV>::TW;
  int lane = threadIdx.x, g = lane >> 4, t = lane & 15;
  int32_t *tr = trl + g * NTT_LDS_GROUP;
  const size_t key = key_idx ? key_idx[task] : task;
  const uint8_t *A = ws.A + kix(ws, task) * K * L * A_POLY;
  g2l_bytes<PP::SIG>(sig + (size_t)task * PP::SIG, sigw, lane);
  if (lane < 2) sigw[PP::SIG / 4 + 1 + lane] = 0;
  wave_sync();
  bool bad = dev_decode_hints<LV>((const uint8_t *)sigw + PP::OFF_H, hm, lane);
  const Tw ftw = ntt_lane_tw(t), itw = intt_lane_tw(t);
  for (int j = g; j < L; j += 4) {
    int32_t x[16];
    load_mask<PP::ZBITS, G1>(x, (const uint8_t *)sigw + PP::OFF_Z + j * PP::ZB, t);
    uint32_t zm = 0;  // |z| < gamma1 - beta, as an offset maximum
#pragma unroll
    for (int r = 0; r < 16; r++) zm = max(zm, (uint32_t)(x[r] + (G1 - BETA - 1)));
    bad |= zm > 2u * (G1 - BETA - 1);
    ntt16(x, ftw, tr, t);
#pragma unroll
    for (int r = 0; r < 16; r++) zh[hat_idx(j, t, r)] = x[r];
  }
  bad = wave_any(bad);
  wave_sync();
  // c t1: two parts of every coefficient, rows g (and g + 4) for the group
  int32_t lo[K > 4 ? 2 : 1][16];
  {
    v4i s[4];
    if (ws.t1s) toep_load(s, ws.t1s + key * TILE_BYTES, lane);
    else toep_load_t1<LV>(s, (const uint32_t *)(pk + key * PP::PK) + 8, lane);
    toep_build(cw, ct, ct + TOEP_WORDS, lane);
    auto half = [&](auto I0c) {
      constexpr int I0 = decltype(I0c)::value;
      v4i acc[8];
      toep_mul<I0, 8>(acc, s, ct, lane);
#pragma unroll
      for (int r = 0; r < 8; r++) {
        lo[0][I0 + r] = acc[r][0] + 32 * acc[r][1];
        if constexpr (K > 4) lo[1][I0 + r] = acc[r][2] + 32 * acc[r][3];
      }
    };
    half(std::integral_constant<int, 0>{});
    __builtin_amdgcn_sched_barrier(0);
    half(std::integral_constant<int, 8>{});
  }
#pragma unroll
  for (int q = 0; q < (K + 3) / 4; q++) {
    const int i = g + 4 * q;
    if (i >= K) break;
    int64_t acc[16];
#pragma unroll
    for (int r = 0; r < 16; r++) acc[r] = 0;
    for (int j = 0; j < L; j++) {
      int32_t a[16];
      load_a(a, A + ((size_t)i * L + j) * A_POLY, t);
#pragma unroll
      for (int r = 0; r < 16; r++) acc[r] += (int64_t)a[r] * zh[hat_idx(j, t, r)];
    }
    int32_t x[16];
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = mont_reduce(acc[r]);
    intt16(x, itw, tr, t);
    int32_t w1[16];
    uint32_t hw[8];
#pragma unroll
    for (int p = 0; p < 8; p++) hw[p] = hm[i * 8 + p];
#pragma unroll
    for (int r = 0; r < 16; r++) {
      int c = t + 16 * r;
      int32_t h = (hw[c >> 5] >> (c & 31)) & 1;
      w1[r] = use_hint<LV>(h, sub_ct1(x[r], lo[q][r]));
    }
    uint32_t vv[16];
    to_consecutive(w1, vv, tr, t);
    pack16_to_lds<PP::W1BITS>(vv, (uint8_t *)w1b + i * PP::W1B, t);
  }
  wave_sync();
  uint32_t *dst = (uint32_t *)(ws.muw1 + (size_t)task * muw1_stride<LV>() + 64);
  for (int w = lane; w < K * PP::W1B / 4; w += 64) dst[w] = w1b[w];
  if (lane == 0) ws.flag[task] = !bad;
}
template <int LV>
__global__ void __launch_bounds__(64, Lv<LV>::K > 4 ? 3 : 4)
    vf_main_k(const uint8_t *pk, const uint32_t *key_idx, const uint8_t *sig, Ws ws, uint32_t count) {
  __shared__ VfLds<LV> lds;
  const uint32_t task = blockIdx.x;
  if (task >= count) return;
  const uint32_t cw = ((const uint32_t *)(ws.cpoly + (size_t)task * N))[threadIdx.x];
  dev_vf_main<LV>(task, cw, lds, pk, key_idx, sig, ws);
}

// ctilde' = H(mu || w1'), verdict; two lanes per task (keccak_pair.h), the
// even lane writing the verdict
template <int LV>
__global__ void __launch_bounds__(256) vf_final_k(const uint8_t *sig, Ws ws, int32_t *verdict, uint32_t count) {
  const uint32_t t = (uint32_t)(((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 1);
  const int half = threadIdx.x & 1;
  if (t >= count) return;  // both lanes of a pair
  const uint8_t *row = ws.muw1 + (size_t)t * muw1_stride<LV>();
  uint32_t a[25];
  shake256_absorb_pair<P<LV>::MUW1>(a, half, [&](int pos) { return *(const uint32_t *)(row + pos + 4 * half); });
  const uint8_t *sg = sig + (size_t)t * P<LV>::SIG;
  uint32_t diff = 0;
#pragma unroll
  for (int w = 0; w < P<LV>::CT / 8; w++) diff |= (uint32_t)load_le_bytes(sg + 8 * w + 4 * half, 4) ^ a[w];
  diff |= pair_swap(diff);
  if (!half) verdict[t] = (ws.flag[t] && diff == 0) ? 1 : 0;
}

// ------------------------------------------------------------------------
// Resident key tables
// ------------------------------------------------------------------------
// t1 as an int8 tile (toeplitz.h) for every key row of a table
template <int LV>
__global__ void __launch_bounds__(64) ks_pk_k(const uint8_t *pk, int8_t *t1s, uint32_t nkeys) {
  const uint32_t key = blockIdx.x;
  if (key >= nkeys) return;
  const int lane = threadIdx.x;
  v4i s[4];
  toep_load_t1<LV>(s, (const uint32_t *)(pk + (size_t)key * P<LV>::PK) + 8, lane);
  int8_t *out = t1s + (size_t)key * TILE_BYTES + (lane & 15) * N + 16 * (lane >> 4);
#pragma unroll
  for (int J = 0; J < 4; J++) *(v4i *)(out + 64 * J) = s[J];
}

// ------------------------------------------------------------------------
// Primitive microbenchmarks
// ------------------------------------------------------------------------
// c_i = INTT(NTT(a_i) o b_i): b read as NTT-domain values; canonical output.
// 256-thread blocks, 16 polynomials per block per iteration, grid-stride.
// PAD = false is the bank-conflicted transpose of the optimisation ablation.
template <bool PAD>
__global__ void __launch_bounds__(256) ntt_mul_k(const int32_t *a, const int32_t *b, int32_t *c, uint64_t count) {
  __shared__ int32_t trl[16 * NTT_LDS_GROUP];
  int g = threadIdx.x >> 4, t = threadIdx.x & 15;
  int32_t *tr = trl + g * NTT_LDS_GROUP;
  const Tw ftw = ntt_lane_tw(t), itw = intt_lane_tw(t);
  for (uint64_t p = (uint64_t)blockIdx.x * 16 + g; p < count; p += (uint64_t)gridDim.x * 16) {
    int32_t x[16], y[16];
    load_strided(x, a + p * N, t);
    load_slots(y, b + p * N, t);
    ntt16<Tw, PAD>(x, ftw, tr, t);
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = mont_mul(x[r], y[r]);
    intt16<Tw, PAD>(x, itw, tr, t);
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = canon(x[r]);
    store_strided(x, c + p * N, t);
  }
}

// ExpandA rejection sampling of one polynomial per lane from a 34-byte input
__global__ void __launch_bounds__(EA_WG) expand_a_seed_k(const uint8_t *seeds, int32_t *out, uint64_t count) {
  uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  __shared__ uint32_t rows[EA_WG / 64][EA_ROWS * EA_ROW];
  const bool valid = p < count;
  const uint8_t *sd = seeds + 34 * (valid ? p : 0);
  uint32_t s[50];
  uint32_t nonce = (uint32_t)sd[32] | ((uint32_t)sd[33] << 8);
  absorb_seed34(s, [&](int pos) { return load_le_bytes(sd + pos, 8); }, nonce);
  const int lane = threadIdx.x & 63;
  expand_a_squeeze_wave<false>(s, (uint8_t *)(out + (p - lane) * N), rows[threadIdx.x >> 6], lane, valid);
}

}  // namespace dil
