// The encrypted matrix product of section IV-E.
#pragma once
#include "ntt_kernels.hpp"

namespace hentt {

// Encrypted element-wise polynomial matrix product (section IV-E), NTT
// domain: C (m x n) += A (m x k) * B (k x n) with ciphertext elements, every
// element product the Mul tensor.  One workgroup per (limb, row i, run of up to
// CT_J columns, tile of 256 coefficients), one coefficient per lane, the run's
// accumulators (three per column) in registers over k.
//
// The words of A are brought to the form of a root power (TwM, 30 instructions
// each) once per run, and every product is then a mul_tw_add: 8 instructions,
// accumulated lazily with no reduction of its own, where a Montgomery product of
// two plain words took 19 and its lazy sum 5 (32 + 60 / columns per element
// product against 83).  Bounds: up to 55 bits A enters below 2q, a product adds
// less than 12.25q (B is canonical: its high word is below 2^23), and 16 steps
// of two products stay below 400q < 512q; the others (FIX) take A canonical (a
// product below 8.25q) and correct after every product (3 + 8.25 < 16; est3
// leaves 33 bits and below alone: 32 products there stay far below 2^(k + 21)).
// Every 16 steps the accumulators are reduced.
//
// Workgroups of one (limb, columns, tile) that differ in the row read the same
// words of B: they are 8 apart in blockIdx, which the dispatcher spreads over
// the 8 XCDs in turn, so that one L2 serves them all.  10 x 9 x 8 elements of
// N = 8192 at 4 limbs: 61.6 us (about half copy rate on A, B and C once each);
// 63.7 with runs of up to 3 columns, 62.3 with 10 (128 VGPRs, and fewer
// workgroups than the chip holds on small matrices); 123 with one column per
// workgroup, Montgomery products and every word of A and B read per product.
constexpr int CT_J = 5;
template <bool FIX> __device__ __forceinline__ TwM ct_word(uint64_t a, const TwM &w30, const TwM &w62, const NttConst &c,
                                                           uint32_t four) {
  uint64_t x = mul_tw(w30, a, c, four), y = mul_tw(w62, a, c, four);
  if constexpr (FIX) {
    x = reduce_word(x, c);
    y = reduce_word(y, c);
  } else {
    x = reduce_est(x, c.nq, c.ce, c.k - 33);
    y = reduce_est(y, c.nq, c.ce, c.k - 33);
  }
  constexpr uint32_t lo = (1u << 30) - 1;
  return TwM{lo32(x) & lo, (uint32_t)(x >> 30), lo32(y) & lo, (uint32_t)(y >> 30)};
}
template <bool FIX> __device__ __forceinline__ uint64_t ct_mac(TwM a, uint64_t b, uint64_t acc, const NttConst &c,
                                                               uint32_t four) {
  const uint64_t s = mul_tw_add(a, b, acc, c, four);
  if constexpr (FIX) return est3(s, c);
  else return s;
}

struct MatmulArgs {
  const uint64_t *A, *B;
  uint64_t *C;
  uint32_t m, n, k, limbs, log_n;
  uint32_t tiles, runs, groups;  // 256-coefficient tiles, column runs, limbs x runs x tiles
};
__global__ __launch_bounds__(256) void k_ct_matmul(MatmulArgs p, const NttConst *__restrict__ lc,
                                                   const MatLimb *__restrict__ ml) {
  uint32_t r = blockIdx.x >> 3;
  const uint32_t i = r % p.m, grp = (r / p.m) * 8 + (blockIdx.x & 7);
  const uint32_t e = (grp % p.tiles) * 256 + threadIdx.x;
  if (grp >= p.groups || e >= (1u << p.log_n)) return;
  r = grp / p.tiles;
  const uint32_t run = r % p.runs, limb = r / p.runs;
  const uint32_t j0 = (uint64_t)run * p.n / p.runs, jn = (run + 1ull) * p.n / p.runs - j0;  // even runs of at most CT_J
  const NttConst c = lc[limb];
  const MatLimb w = ml[limb];
  const uint64_t P = (uint64_t)p.limbs << p.log_n;
  const uint64_t off = ((uint64_t)limb << p.log_n) + e;
  const uint64_t *a = p.A + (uint64_t)i * p.k * 2 * P + off;
  const uint64_t *b = p.B + (uint64_t)j0 * 2 * P + off;
  uint64_t *cc = p.C + ((uint64_t)i * p.n + j0) * 3 * P + off;
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    constexpr bool FIX = decltype(FX)::value;
    const uint32_t four = opaque4();
    uint64_t acc[CT_J][3];
    static_for<0, CT_J>([&](auto J) __attribute__((always_inline)) {
      constexpr int j = decltype(J)::value;
      if (j < (int)jn) {
#pragma unroll
        for (int s = 0; s < 3; ++s) acc[j][s] = cc[(uint64_t)(3 * j + s) * P];
      }
    });
#pragma unroll 1
    for (uint32_t l0 = 0; l0 < p.k; l0 += 16) {
      const uint32_t l1 = l0 + 16 < p.k ? l0 + 16 : p.k;
#pragma unroll 1
      for (uint32_t l = l0; l < l1; ++l) {
        const uint64_t *al = a + (uint64_t)l * 2 * P, *bl = b + (uint64_t)l * p.n * 2 * P;
        uint64_t bv[CT_J][2];
        static_for<0, CT_J>([&](auto J) __attribute__((always_inline)) {
          constexpr int j = decltype(J)::value;
          if (j < (int)jn) {
            bv[j][0] = bl[(uint64_t)(2 * j) * P];
            bv[j][1] = bl[(uint64_t)(2 * j + 1) * P];
          }
        });
        const TwM a0 = ct_word<FIX>(al[0], w.w30, w.w62, c, four), a1 = ct_word<FIX>(al[P], w.w30, w.w62, c, four);
        static_for<0, CT_J>([&](auto J) __attribute__((always_inline)) {
          constexpr int j = decltype(J)::value;
          if (j < (int)jn) {
            acc[j][0] = ct_mac<FIX>(a0, bv[j][0], acc[j][0], c, four);
            acc[j][1] = ct_mac<FIX>(a1, bv[j][0], ct_mac<FIX>(a0, bv[j][1], acc[j][1], c, four), c, four);
            acc[j][2] = ct_mac<FIX>(a1, bv[j][1], acc[j][2], c, four);
          }
        });
      }
      static_for<0, CT_J>([&](auto J) __attribute__((always_inline)) {
        constexpr int j = decltype(J)::value;
        if (j < (int)jn) {
#pragma unroll
          for (int s = 0; s < 3; ++s) acc[j][s] = reduce_word(acc[j][s], c);
        }
      });
    }
    static_for<0, CT_J>([&](auto J) __attribute__((always_inline)) {
      constexpr int j = decltype(J)::value;
      if (j < (int)jn) {
#pragma unroll
        for (int s = 0; s < 3; ++s) cc[(uint64_t)(3 * j + s) * P] = acc[j][s];
      }
    });
  });
}

}  // namespace hentt
