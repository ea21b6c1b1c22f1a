// Relinearization (Relin of section II-A) with the RNS digit key switch:
//   c' = (c0, c1) + round(P^-1 sum_j [c2]_{q_j} evk_j)  mod q,
// over the ciphertext primes q_0 .. q_{l-1} extended by a special prime P.
// The digits d_j = INTT_j(c2_j) are integers in [0, q_j).  For every target
// prime q_t (t <= l) each digit is reduced modulo q_t and forward-transformed
// (the reduction fused into the transform's first load), and the products
// with the key-switching key are accumulated in registers over the digits
// (fused into the transform's last stage):
//   acc_s[t] = sum_j NTT_t(d_j mod q_t) . ksk[j][s][t]   (s = 0, 1).
// The products are Montgomery products (off by 2^-60, see ks_mac) on the
// lazy transform outputs, summed lazily; one product by the inverse factor per
// output word removes it before the store.  The same
// epilogue adds P c_s (s = 0, 1) for t < l: round((x + P c_s) / P) =
// c_s + round(x / P) exactly (x and x + P c_s agree mod P), so the rescale
// of rescale_kernels.hpp that divides by P with rounding also completes
// c' = (c0, c1) + round(P^-1 c2 evk).
#pragma once
#include "ntt_kernels.hpp"

namespace hentt {

struct KsLimb {     // per target prime q_t of one level
  TwM r, pm;        // 2^60 mod q_t, P mod q_t (t < l)
  uint64_t mu;      // floor(2^64 / q_t)
};

struct KsArgs {
  const uint64_t *d;    // [batch][l][N] digits, coefficient domain, canonical mod q_j, or,
                        // two-pass sizes, behind the inverse transform's block pass
  const uint64_t *ksk;  // [l][2][l + 1][N] NTT domain
  uint64_t *e;          // [batch][l][l + 1][N] column-pass scratch (two-pass sizes)
  uint64_t *acc;        // [batch][2][l + 1][N]
  const uint64_t *c;    // [batch][3][l][N] NTT domain: (c0, c1) enter as P c_s
  const KsLimb *kc;     // [l + 1]
  uint64_t *part;       // [splits][batch][2][l + 1][N] partial sums when splits > 1
  uint32_t batch, l;
  uint32_t splits;      // workgroups a block's digits are spread over
  uint32_t col_splits;  // workgroups a digit's column tile spreads its target primes over
};

// A digit word x < q_j < 2^60 as an input of the transform modulo q_t: as it is
// (the forward transform takes any 60-bit word, see rs_prologue), except that
// moduli of 33 or fewer bits reduce it into [0, 2 q_t) (the estimate
// floor(x mu / 2^64) of x / q_t is short by at most one).
__device__ __forceinline__ uint64_t ks_lift(uint64_t x, uint64_t mu, const NttConst &c) {
  if (c.k < 34) x -= mulhi64(x, mu) * c.q;
  return x;
}

// acc0 += v . key0 2^-60, acc1 += v . key1 2^-60 (mod q, mont30_mul_add) for the
// words of v (lazy forward outputs) held in the (0, E) map of a 2^B block; key0 at
// k, key1 one prime-row further (`row` blocks of 2^B words); j counts the digits.
// The accumulators by modulus size:
//   34..55 bits  less than 5q a digit, cut back (est3) every 32 digits: below
//                3q + 160q < 2^63;
//   56..60 bits  cut back ahead of every digit: below 3q + 7q (the key, canonical,
//                is the factor below q);
//   33 or fewer  never cut back: below 5q 2^12, for the most limbs there can be.
// The two products run one after the other (scheduling barrier) so that only one
// key array is live.
template <int B, int E, bool FIX>
__device__ __forceinline__ void ks_mac(uint64_t (&v)[1 << E], const uint64_t *k, uint32_t row, uint32_t lp,
                                       uint64_t (&acc0)[1 << E], uint64_t (&acc1)[1 << E], const NttConst &c,
                                       uint32_t j) {
  uint64_t kv[1 << E];
  load_global<B, E, 0, E>(kv, k, lp);
  const uint32_t four = opaque4();
  if (FIX || (j & 31) == 31) {
#pragma unroll
    for (int s = 0; s < (1 << E); ++s) {
      acc0[s] = est3(acc0[s], c);
      acc1[s] = est3(acc1[s], c);
    }
  }
  reduce_for_mont<E, FIX>(v, c);
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) {
    if constexpr (FIX) acc0[s] = mont30_mul_add(split30(kv[s]), v[s], acc0[s], c, four);
    else acc0[s] = mont30_mul_add(split30(v[s]), kv[s], acc0[s], c, four);
  }
  __builtin_amdgcn_sched_barrier(0);
  load_global<B, E, 0, E>(kv, k + ((uint64_t)row << B), lp);
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) {
    if constexpr (FIX) acc1[s] = mont30_mul_add(split30(kv[s]), v[s], acc1[s], c, four);
    else acc1[s] = mont30_mul_add(split30(v[s]), kv[s], acc1[s], c, four);
  }
}

// Accumulators (sums of Montgomery products) to canonical values: times 2^60, plus P c_s when cs (c_s's words of the block, in the (0, E)
// map) is given; est3 keeps the sum of the two products (12q each) below 16q.
template <int B, int E>
__device__ __forceinline__ void ks_finish(uint64_t (&acc)[1 << E], const KsLimb &kc, const NttConst &c,
                                          const uint64_t *cs, uint32_t lp) {
  const uint32_t four = opaque4();
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) acc[s] = mul_tw(kc.r, acc[s], c, four);
  if (cs) {
    uint64_t cv[1 << E];
    load_global<B, E, 0, E>(cv, cs, lp);
#pragma unroll
    for (int s = 0; s < (1 << E); ++s) acc[s] = mul_tw_add(kc.pm, cv[s], est3(acc[s], c), c, four);
  }
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) acc[s] = reduce_word(acc[s], c);
}

// Digit t modulo its own prime, back in the NTT domain, is c2's limb t itself: at
// j = t the kernels read that (canonical words, in the (0, E) map) and transform
// nothing, one transform in l + 1 (2^15, 8 primes, 32 entries, the whole
// relinearization: 686 us without, 671 with).
__device__ __forceinline__ const uint64_t *ks_own(const KsArgs &a, uint32_t b, uint32_t t, int logn, uint32_t off) {
  return a.c + ((((uint64_t)b * 3 + 2) * a.l + t) << logn) + off;
}

// c_s's words (s = 0, 1) at block offset `off` of target prime t for batch
// entry b, or null for the special prime (t = l).
__device__ __forceinline__ const uint64_t *ks_cs(const KsArgs &a, uint32_t b, uint32_t s, uint32_t t, int logn,
                                                 uint32_t off) {
  return t < a.l ? a.c + ((((uint64_t)b * 3 + s) * a.l + t) << logn) + off : nullptr;
}

// Whole transforms (N <= 2^12, up to 512 lanes): one workgroup per (batch entry,
// target prime), looping over the digits.
template <int LOGN, int E>
__global__ __launch_bounds__(1 << (LOGN - E)) void k_ks_whole(KsArgs a, const TwM *__restrict__ tw,
                                                               const NttConst *__restrict__ lc) {
  __shared__ uint64_t lds[LdsSize<LOGN>::value];
  const uint32_t L1 = a.l + 1;
  const uint32_t t = blockIdx.x / a.batch, b = blockIdx.x % a.batch;
  const NttConst c = lc[t];
  const KsLimb kc = a.kc[t];
  const TwM *tt = tw + (size_t)t * 2 * (1u << LOGN);
  const uint32_t tid = threadIdx.x;
  using F = FwdFirst<LOGN, E>;
  using M0 = RoundMap<LOGN, E, 0, E>;
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    constexpr bool FIX = decltype(FX)::value;
    uint64_t acc0[1 << E], acc1[1 << E];
  #pragma unroll
    for (int s = 0; s < (1 << E); ++s) acc0[s] = acc1[s] = 0;
  #pragma unroll 1
    for (uint32_t j = 0; j < a.l; ++j) {
      if (j > 0) __syncthreads();  // the previous digit's last LDS reads are done
      uint64_t v[1 << E];
      if (j == t) {
        load_global<LOGN, E, 0, E>(v, ks_own(a, b, t, LOGN, 0), M0::lane_part(tid));
      } else {
        load_global<LOGN, E, F::LO, F::R>(v, a.d + (((uint64_t)b * a.l + j) << LOGN),
                                           RoundMap<LOGN, E, F::LO, F::R>::lane_part(tid));
#pragma unroll
        for (int s = 0; s < (1 << E); ++s) v[s] = ks_lift(v[s], kc.mu, c);
        // an opaque copy of the table pointer per digit: the twiddles (the same
        // for every digit) are re-read from cache instead of held in VGPRs
        fwd_block_rounds<LOGN, E, F::LO, F::R, FIX>(v, LOGN, lds, tid, 0, opaque(tt), c);
      }
      ks_mac<LOGN, E, FIX>(v, a.ksk + (((uint64_t)j * 2 * L1 + t) << LOGN), L1, M0::lane_part(tid), acc0, acc1, c,
                           j);
    }
    ks_finish<LOGN, E>(acc0, kc, c, ks_cs(a, b, 0, t, LOGN, 0), M0::lane_part(tid));
    store_global_m0<LOGN, E>(acc0, a.acc + (((uint64_t)b * 2 * L1 + t) << LOGN), lds, tid);
    ks_finish<LOGN, E>(acc1, kc, c, ks_cs(a, b, 1, t, LOGN, 0), M0::lane_part(tid));
    store_global_m0<LOGN, E>(acc1, a.acc + (((uint64_t)(b * 2 + 1) * L1 + t) << LOGN), lds, tid);
  });
}

// Two-pass sizes, pass 1: for a tile of columns of digit j, the last EC inverse
// stages of the digit (the words behind the block pass), which end in the lane map
// the forward pass begins with, so that the coefficients stay in registers; then,
// per target prime of this workgroup's run, the first EC forward stages modulo q_t
// into e.  It writes l words per word read, so a forward pass of its own per
// prime, reading the digit back each time, was bound by those reads: N = 2^15, 8
// primes, 32 entries, 180 us with streaming loads, 147 with ordinary ones, and 40 of
// the inverse column pass; 130 together.  Four waves per SIMD (128 registers).
template <int LOGN, int EC>
__global__ __launch_bounds__(cols_lanes<EC>(), EC < 8 ? 4 : 1) void k_ks_cols(KsArgs a, const TwM *__restrict__ tw,
                                                              const NttConst *__restrict__ lc) {
  __shared__ uint64_t lds[cols_lds<EC>()];
  constexpr uint32_t tiles = cols_blocks_per_unit<LOGN, EC>();
  const uint32_t L1 = a.l + 1;
  uint32_t r = blockIdx.x / tiles;
  const uint32_t col = (blockIdx.x % tiles) * LC<EC> + threadIdx.x % LC<EC>;
  const uint32_t part = r % a.col_splits;
  r /= a.col_splits;
  const uint32_t j = r % a.l, b = r / a.l;
  const uint64_t *src = a.d + (((uint64_t)b * a.l + j) << LOGN);
  uint64_t *dst = a.e + (((uint64_t)b * a.l + j) * L1 << LOGN);
  uint64_t x[16];
  {
    const NttConst c = lc[j];
    by_class(c, [&](auto FX) __attribute__((always_inline)) {
      lcol_inv<LOGN, EC, decltype(FX)::value>(
          x, [&](uint32_t row) { return gload<false>(src, (row << (LOGN - EC)) + col); },
          tw + ((size_t)j * 2 + 1) * (1u << LOGN), c, lds);
    });
  }
  const uint32_t t1 = (part + 1) * L1 / a.col_splits;
#pragma unroll 1
  for (uint32_t t = part * L1 / a.col_splits; t < t1; ++t) {
    if (t == j) continue;  // ks_own
    __syncthreads();       // the last LDS reads before this prime's writes
    const NttConst c = lc[t];
    const uint64_t mu = a.kc[t].mu;
    uint64_t *o = dst + ((uint64_t)t << LOGN);
    by_class(c, [&](auto FX) __attribute__((always_inline)) {
      uint64_t v[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = ks_lift(x[k], mu, c);
      lcol_fwd<LOGN, EC, decltype(FX)::value>(
          v, [&](uint32_t row, uint64_t y) { gstore<true>(o, (row << (LOGN - EC)) + col, y); },
          tw + (size_t)t * 2 * (1u << LOGN), c, lds);
    });
  }
}

// Two-pass sizes, pass 2: per (batch entry, target prime, block), the block
// rounds of every digit, accumulated with the key in registers.  300 to 320 us, VALU
// busy 60% of a counter run; its 0.93 GB take 190 at the copy rate.  At N = 2^15, 8 primes, 32 entries, the
// whole relinearization: 720 us with Montgomery products of 64-bit words, 690 with
// mont30_mul at the 134 VGPRs it takes (three waves per SIMD), 678 held to 128
// (four waves), 600 with the column passes fused.  The key in root-power form, a third fewer
// instructions than the 64-bit products for twice its bytes, gave 716.  A small batch
// has fewer blocks than the chip has places for waves; their digits are then
// spread over `splits` workgroups, whose partial sums k_ks_sum adds up.
template <int LOGN, int ST, int B, int E>
__global__ __launch_bounds__(1 << (B - E), 4) void k_ks_blocks(KsArgs a, const TwM *__restrict__ tw,
                                                             const NttConst *__restrict__ lc) {
  __shared__ uint64_t lds[LdsSize<B>::value];
  constexpr uint32_t tiles = 1u << (LOGN - B);
  const uint32_t L1 = a.l + 1;
  const uint32_t tile = blockIdx.x % tiles, blockStart = tile << B;
  uint32_t r = blockIdx.x / tiles;
  const uint32_t b = r % a.batch;
  r /= a.batch;
  const uint32_t t = r % L1, part = r / L1;
  const uint32_t j0 = part * a.l / a.splits, j1 = (part + 1) * a.l / a.splits;
  const NttConst c = lc[t];
  const KsLimb kc = a.kc[t];
  const TwM *tt = tw + (size_t)t * 2 * (1u << LOGN);
  const uint32_t tid = threadIdx.x;
  using F = FwdFirst<ST, E>;
  using M0 = RoundMap<B, E, 0, E>;
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    constexpr bool FIX = decltype(FX)::value;
    uint64_t acc0[1 << E], acc1[1 << E];
#pragma unroll
    for (int s = 0; s < (1 << E); ++s) acc0[s] = acc1[s] = 0;
#pragma unroll 1
    for (uint32_t j = j0; j < j1; ++j) {
      if (j > j0) __syncthreads();  // the previous digit's last LDS reads are done
      uint64_t v[1 << E];
      if (j == t) {
        load_global<B, E, 0, E>(v, ks_own(a, b, t, LOGN, blockStart), M0::lane_part(tid));
      } else {
        load_global<B, E, F::LO, F::R>(v, a.e + ((((uint64_t)b * a.l + j) * L1 + t) << LOGN) + blockStart,
                                       RoundMap<B, E, F::LO, F::R>::lane_part(tid));
        fwd_block_rounds<B, E, F::LO, F::R, FIX>(v, LOGN, lds, tid, blockStart, opaque(tt), c);
      }
      ks_mac<B, E, FIX>(v, a.ksk + (((uint64_t)j * 2 * L1 + t) << LOGN) + blockStart, L1 << (LOGN - B), M0::lane_part(tid),
                   acc0, acc1, c, j - j0);
    }
    const uint64_t o0 = (((uint64_t)b * 2 * L1 + t) << LOGN) + blockStart, o1 = o0 + ((uint64_t)L1 << LOGN);
    uint64_t *out = a.acc;
    if (a.splits > 1) {
      out = a.part + ((uint64_t)part * a.batch * 2 * L1 << LOGN);
    } else {
      ks_finish<B, E>(acc0, kc, c, ks_cs(a, b, 0, t, LOGN, blockStart), M0::lane_part(tid));
      ks_finish<B, E>(acc1, kc, c, ks_cs(a, b, 1, t, LOGN, blockStart), M0::lane_part(tid));
    }
    store_global_m0<B, E>(acc0, out + o0, lds, tid);
    store_global_m0<B, E>(acc1, out + o1, lds, tid);
  });
}

// Adds up the partial sums (ks_mac's accumulators) of k_ks_blocks and
// finishes them as it does.  One lane per word of [batch][2][l + 1][N].
template <int LOGN> __global__ __launch_bounds__(256) void k_ks_sum(KsArgs a, const NttConst *__restrict__ lc) {
  constexpr uint32_t tiles = 1u << (LOGN - 8);
  const uint32_t L1 = a.l + 1, row = blockIdx.x / tiles;  // (b, s, t), t fastest
  const uint32_t t = row % L1, s = (row / L1) & 1, b = row / (2 * L1);
  const uint32_t i = (blockIdx.x % tiles) * 256 + threadIdx.x;
  const uint64_t words = (uint64_t)a.batch * 2 * L1 << LOGN, at = ((uint64_t)row << LOGN) + i;
  const NttConst c = lc[t];
  const KsLimb kc = a.kc[t];
  const uint32_t four = opaque4();
  uint64_t x = est3(a.part[at], c);
  for (uint32_t k = 1; k < a.splits; ++k) x = est3(x + a.part[k * words + at], c);
  x = mul_tw(kc.r, x, c, four);
  const uint64_t *cs = ks_cs(a, b, s, t, LOGN, i);
  if (cs) x = mul_tw_add(kc.pm, *cs, est3(x, c), c, four);
  a.acc[at] = reduce_word(x, c);
}

}  // namespace hentt
