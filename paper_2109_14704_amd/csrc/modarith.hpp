// 64-bit modular arithmetic for gfx950 built from 32-bit multiplies.
//
// gfx950 has no 64x64 multiplier; v_mad_u64_u32 (32x32+64 -> 64) and
// v_mul_hi_u32 issue at full VALU rate, so every 64-bit product below is
// spelled as 32-bit partial products the compiler maps onto those
// instructions (the paper's mul_low_high lesson, section III-A-2, restated
// for this ISA).  Moduli satisfy q < 2^60 (so 16q < 2^64).
#pragma once
#include <stdint.h>

#include "records.hpp"
#ifdef HENTT_HOST_TEST
// Host build of this header for the CPU property tests of the arithmetic.
#define __device__
#define __forceinline__ inline
static inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
#else
#include <hip/hip_runtime.h>
#endif

namespace hentt {

__device__ __forceinline__ uint32_t lo32(uint64_t x) { return (uint32_t)x; }
__device__ __forceinline__ uint32_t hi32(uint64_t x) { return (uint32_t)(x >> 32); }
__device__ __forceinline__ uint64_t mad32(uint32_t a, uint32_t b, uint64_t c) { return (uint64_t)a * b + c; }

// floor(a*b / 2^64), exact.
__device__ __forceinline__ uint64_t mulhi64(uint64_t a, uint64_t b) {
  uint32_t a0 = lo32(a), a1 = hi32(a), b0 = lo32(b), b1 = hi32(b);
  uint64_t m1 = mad32(a1, b0, __umulhi(a0, b0));
  uint64_t m2 = mad32(a0, b1, lo32(m1));
  return mad32(a1, b1, hi32(m1)) + hi32(m2);
}

// Full 128-bit product a*b as (hi, lo).
__device__ __forceinline__ void mul128(uint64_t a, uint64_t b, uint64_t& hi, uint64_t& lo) {
  uint32_t a0 = lo32(a), a1 = hi32(a), b0 = lo32(b), b1 = hi32(b);
  uint64_t p00 = mad32(a0, b0, 0);
  uint64_t m1 = mad32(a1, b0, hi32(p00));
  uint64_t m2 = mad32(a0, b1, lo32(m1));
  lo = ((uint64_t)lo32(m2) << 32) | lo32(p00);
  hi = mad32(a1, b1, hi32(m1)) + hi32(m2);
}

// Quotient estimate for Shoup's product: floor(W' Y / 2^64) minus 0, 1 or 2.
// Only the three high partial products enter (a1 b1 and the high halves of
// the cross products); the low product a0 b0 and the low halves of the
// cross products, which together carry less than 3 into bit 64, are dropped.
// Three multiplies instead of four, and no carry chain.
__device__ __forceinline__ uint64_t shoup_q(uint64_t Ws, uint64_t Y) {
  const uint32_t a0 = lo32(Ws), a1 = hi32(Ws), b0 = lo32(Y), b1 = hi32(Y);
  const uint64_t s = (uint64_t)__umulhi(a1, b0) + __umulhi(a0, b1);
  return mad32(a1, b1, s);
}

// Shoup product (Harvey 2014, the butterfly of Algorithm 1 in section III-B):
// W Y mod q up to a multiple of q, W' = floor(W 2^64 / q), nq = -q mod 2^64.
// With the estimate above the result lies in [0, 4q) for any Y < 2^64
// (exact quotient: [0, 2q); each missing unit of the quotient adds q).
__device__ __forceinline__ uint64_t shoup(uint64_t W, uint64_t Ws, uint64_t Y, uint64_t nq) {
  return W * Y + shoup_q(Ws, Y) * nq;  // = W Y - Q q  (mod 2^64)
}

// x >= m ? x - m : x, given nm = -m mod 2^64 (one 64-bit add, one compare).
__device__ __forceinline__ uint64_t csubn(uint64_t x, uint64_t nm) {
  const uint64_t d = x + nm;
  return d < x ? d : x;
}
__device__ __forceinline__ uint64_t csub(uint64_t x, uint64_t m) { return x >= m ? x - m : x; }

// Forward (Cooley-Tukey) lazy butterfly, Algorithm 1 with a wider lazy range:
// X, Y in [0, 8q) on entry and exit (q < 2^60); X' = X + W Y, Y' = X - W Y
// (mod q).  X is brought below 4q, T = W Y mod q lies in [0, 4q), so X + T and
// X - T + 4q stay in [0, 8q).
__device__ __forceinline__ void ct_bfly(uint64_t &X, uint64_t &Y, uint64_t W, uint64_t Ws, const ModQ &m) {
  const uint64_t x = csubn(X, m.nq4);
  const uint64_t T = shoup(W, Ws, Y, m.nq);
  X = x + T;
  Y = (x + m.q4) - T;
}

// Forward butterfly of the design ladder's register rounds, with the correction
// of X taken every second stage: values lie in [0, 16q) (q < 2^60, so 16q < 2^64).
// CORR: X (below 16q) is first brought below 8q, and the outputs lie below
// 12q; otherwise X must already be below 12q and the outputs lie below 16q.
// A pass corrects at its even-numbered stages (the first one included), so
// two uncorrected stages never follow each other and a pass may start from
// any values below 16q.  T lies in [0, 4q) for any Y < 2^64.
template <bool CORR>
__device__ __forceinline__ void ct_bfly16(uint64_t &X, uint64_t &Y, uint64_t W, uint64_t Ws, const ModQ &m) {
  uint64_t x = X;
  if constexpr (CORR) x = csubn(X, m.nq4 + m.nq4);  // -8q mod 2^64
  const uint64_t T = shoup(W, Ws, Y, m.nq);
  X = x + T;
  Y = (x + m.q4) - T;
}

// Inverse (Gentleman-Sande) lazy butterfly after Harvey: X, Y in [0, 4q) on
// entry and exit; X' = X + Y, Y' = W (X - Y) (mod q).  The counterpart of ct_bfly for
// an inverse with Shoup products; the library's inverse is gs_bfly_m.
__device__ __forceinline__ void gs_bfly(uint64_t &X, uint64_t &Y, uint64_t W, uint64_t Ws, const ModQ &m) {
  const uint64_t s = X + Y;
  const uint64_t d = (X + m.q4) - Y;
  X = csubn(s, m.nq4);
  Y = shoup(W, Ws, d, m.nq);
}

// Canonical reductions: from [0, 8q) and from [0, 4q) to [0, q).
__device__ __forceinline__ uint64_t reduce_8q(uint64_t x, const ModQ &m) {
  return csubn(csubn(csubn(x, m.nq4), m.nq2), m.nq);
}
__device__ __forceinline__ uint64_t reduce_4q(uint64_t x, const ModQ &m) { return csubn(csubn(x, m.nq2), m.nq); }
// From [0, 16q) (forward outputs of ct_bfly16 passes) to [0, q).
__device__ __forceinline__ uint64_t reduce_16q(uint64_t x, const ModQ &m) {
  return csubn(csubn(csubn(csubn(x, m.nq4 + m.nq4), m.nq4), m.nq2), m.nq);
}

// Any x < 2^64 to [0, 2q) by a quotient estimate, for q > 2^33 (bit length
// k >= 34), with c = floor(2^(k+31) / q) (below 2^32) and sh = k - 33:
// e = floor(hi32(x) c / 2^(k-1)) never exceeds x / q and falls short of it
// by less than 2 (the low word of x weighs less than 2^32 / q < 1/2, the
// truncation of c less than hi32(x) / 2^(k-1) < 1/2, the floor less than 1),
// so x - e q lies in [0, 2q).  One multiply-high, a shift and the 32 x 64-bit
// product e q, against a chain of conditional subtractions.
__device__ __forceinline__ uint64_t reduce_est(uint64_t x, uint64_t nq, uint32_t c, uint32_t sh) {
  const uint32_t e = __umulhi(hi32(x), c) >> sh;
  // x - e q (mod 2^64): the low product in the multiply-add's accumulator,
  // e times the high word of -q added to the high word alone
  const uint64_t r = mad32(e, lo32(nq), x);
  uint32_t t = e * hi32(nq);
#ifndef HENTT_HOST_TEST
  // kept a plain multiply and add: fused into one more 32x32+64 multiply-add
  // it costs two register moves
  asm("" : "+v"(t));
#endif
  return ((uint64_t)(hi32(r) + t) << 32) | lo32(r);
}
// c of reduce_est from the Barrett constant mu = floor(2^(2k) / q):
// floor(mu / 2^(k-31)) = floor(2^(k+31) / q).
__device__ __forceinline__ uint32_t est_c(uint64_t mu, uint32_t k) { return (uint32_t)(mu >> (k - 31)); }

// ---------------------------------------------------------------------------
// Products by a root power, in the transforms' form (TwM).  With Y = y1 2^32 +
// y0, A = W 2^30 mod q and B = W 2^62 mod q,
//   z = A y0 + B y1 = W Y 2^30 (mod q),
// and one Montgomery step (Montgomery 1985) with a 32-bit multiplier divides
// by 2^30: split at bit 30, z + m q = p0 + 2^30 p1 with
//   p0 = a0 y0 + b0 y1 + m qlo < 3 2^62,   p1 = a1 y0 + b1 y1 + m qhi,
// and m = -p0 qlo^-1 mod 2^32 clears the low 32 bits of p0, so that
// (z + m q) / 2^30 = p1 + 4 hi32(p0) exactly.  The result T = W Y mod q lies in
// [0, 12q) for any Y < 2^64 (three terms below q 2^32 over 2^30).  Splitting at
// 30 bits is what keeps p0 inside one 64-bit accumulator: no carry between the
// halves, so all of it is seven multiply-adds and one low product, and X + T
// costs nothing more (X starts p1).  A Shoup product takes nine multiplies
// and about four additions more.  In registers at full occupancy (the issue-rate
// microbenchmarks): 3250 G forward and 3120 G inverse butterflies a second, 1917 G
// with Shoup products.
//
// The last multiply-add's factor is an opaque 4: spelled as a shift it would
// cost two register moves and an add.
__device__ __forceinline__ uint32_t opaque4() {
#ifdef HENTT_HOST_TEST
  return 4;
#else
  uint32_t f;
  asm("s_mov_b32 %0, 4" : "=s"(f));
  return f;
#endif
}
// x + W y mod q, short of 12q above x.
__device__ __forceinline__ uint64_t mul_tw_add(TwM w, uint64_t y, uint64_t x, const NttConst &c, uint32_t four) {
  const uint32_t y0 = lo32(y), y1 = hi32(y);
  uint64_t p0 = mad32(w.a0, y0, 0);
  p0 = mad32(w.b0, y1, p0);
  uint64_t p1 = mad32(w.a1, y0, x);
  p1 = mad32(w.b1, y1, p1);
  const uint32_t m = lo32(p0) * c.qi;
  p0 = mad32(m, c.qlo, p0);
  p1 = mad32(m, c.qhi, p1);
  return mad32(hi32(p0), four, p1);
}
__device__ __forceinline__ uint64_t mul_tw(TwM w, uint64_t y, const NttConst &c, uint32_t four) {
  return mul_tw_add(w, y, 0, c, four);
}

// Any x < 2^64 to [0, 3q) for q > 2^33, by the quotient estimate
// floor(hi32(x) floor(2^64 / q) / 2^32): short of x / q by less than 2.5 (the
// floor, the truncated constant and the dropped low word: 1 + 1 + 1/2).  Four
// instructions, as many as one conditional subtraction.
__device__ __forceinline__ uint64_t est3(uint64_t x, const NttConst &c) {
  const uint32_t e = __umulhi(hi32(x), c.c64);
  const uint64_t r = mad32(e, lo32(c.nq), x);
  uint32_t t = e * hi32(c.nq);
#ifndef HENTT_HOST_TEST
  asm("" : "+v"(t));  // kept a plain multiply and add, as in reduce_est
#endif
  return ((uint64_t)(hi32(r) + t) << 32) | lo32(r);
}

// Canonical form of a lazy word, any modulus, with the estimate's 32 bits taken
// from x >> s0 and e = floor((x >> s0) ce / 2^32) >> s1:
//   k >= 34: s0 = 32, s1 = k - 33, reduce_est's estimate of any x < 2^64;
//   smaller: s0 = max(0, k - 11), s1 = k - 1 - s0, for x < 2^(k + 21), the
//            lazy bound of either transform.
__device__ __forceinline__ uint64_t reduce_word(uint64_t x, const NttConst &c) {
  const uint32_t e = __umulhi((uint32_t)(x >> c.s0), c.ce) >> c.s1;
  const uint64_t r = mad32(e, lo32(c.nq), x);
  uint32_t t = e * hi32(c.nq);
#ifndef HENTT_HOST_TEST
  asm("" : "+v"(t));
#endif
  return csubn(((uint64_t)(hi32(r) + t) << 32) | lo32(r), c.nq);
}

// Forward (Cooley-Tukey) butterfly: X' = X + W Y, Y' = X - W Y + 12q (mod q);
// both below X + 12q.  Eleven instructions.  X must leave room for 12q below
// 2^64; Y is any 64-bit word.  Which stages correct X first: schedule.hpp.
__device__ __forceinline__ void ct_bfly_m(uint64_t &X, uint64_t &Y, TwM w, const NttConst &c, uint32_t four) {
  const uint64_t s = mul_tw_add(w, Y, X, c, four);
  Y = ((X << 1) + c.off) - s;
  X = s;
}

// Inverse (Gentleman-Sande) butterfly: X' = X + Y, Y' = W (X - Y) below 12q;
// off is a multiple of q at least as large as Y, and X + off < 2^64.
__device__ __forceinline__ void gs_bfly_m(uint64_t &X, uint64_t &Y, TwM w, uint64_t off, const NttConst &c,
                                          uint32_t four) {
  const uint64_t d = (X + off) - Y;
  X = X + Y;
  Y = mul_tw(w, d, c, four);
}

// Barrett reduction of a 128-bit z < 2^(2k+1) modulo q, 2^(k-1) <= q < 2^k
// (k <= 60), with mu = floor(2^(2k) / q): quotient estimate
// floor(floor(z / 2^(k-1)) * mu / 2^(k+1)) is short by at most 3.
__device__ __forceinline__ uint64_t barrett(uint64_t zhi, uint64_t zlo, uint64_t q, uint64_t mu, uint32_t k) {
  // z1 = z >> (k-1), fits in 64 bits since z < 2^(2k+1) and k <= 60
  uint32_t sh = k - 1;
  uint64_t z1 = (zlo >> sh) | (zhi << (64 - sh));
  uint64_t ph, pl;
  mul128(z1, mu, ph, pl);
  uint32_t sh2 = k + 1;
  uint64_t q3 = (pl >> sh2) | (ph << (64 - sh2));
  uint64_t r = zlo - q3 * q;
  r = csub(r, q);
  r = csub(r, q);
  r = csub(r, q);
  return r;
}

// a * b mod q for canonical a, b.
__device__ __forceinline__ uint64_t mulmod(uint64_t a, uint64_t b, uint64_t q, uint64_t mu, uint32_t k) {
  uint64_t h, l;
  mul128(a, b, h, l);
  return barrett(h, l, q, mu, k);
}

// (a*b + c*d) mod q with a single reduction (mad_mod, section III-A-1).
__device__ __forceinline__ uint64_t madmod(uint64_t a, uint64_t b, uint64_t c, uint64_t d, uint64_t q, uint64_t mu,
                                           uint32_t k) {
  uint64_t h1, l1, h2, l2;
  mul128(a, b, h1, l1);
  mul128(c, d, h2, l2);
  uint64_t l = l1 + l2;
  uint64_t h = h1 + h2 + (l < l1 ? 1 : 0);
  return barrett(h, l, q, mu, k);
}

// Montgomery reduction (Montgomery 1985) with R = 2^64, for the products
// whose factor R^-1 is cancelled elsewhere (folded into the N^-1 scaling of
// the inverse transform that follows them).  For T = hi 2^64 + lo < q R and
// qinv = -q^-1 mod 2^64, m = lo qinv mod 2^64 makes T + m q a multiple of R;
// its low word is zero, with a carry out exactly when lo != 0, so
// (T + m q) / R = hi + floor(m q / 2^64) + [lo != 0], which is T R^-1 mod q
// in [0, 2q).  Two half products (a low one, a high one) and no correction
// steps, where Barrett takes a full 128-bit product, a low product, two
// variable shifts and three conditional subtractions.
__device__ __forceinline__ uint64_t redc(uint64_t hi, uint64_t lo, uint64_t q, uint64_t qinv) {
  const uint64_t m = lo * qinv;
  return hi + mulhi64(m, q) + (lo != 0 ? 1 : 0);
}
// a b R^-1 mod q in [0, 2q) for a b < q R.
__device__ __forceinline__ uint64_t mont_mul(uint64_t a, uint64_t b, uint64_t q, uint64_t qinv) {
  uint64_t h, l;
  mul128(a, b, h, l);
  return redc(h, l, q, qinv);
}
// (a b + c d) R^-1 mod q in [0, 2q) for a b + c d < q R (one reduction).
__device__ __forceinline__ uint64_t mont_mad(uint64_t a, uint64_t b, uint64_t c, uint64_t d, uint64_t q,
                                            uint64_t qinv) {
  uint64_t h1, l1, h2, l2;
  mul128(a, b, h1, l1);
  mul128(c, d, h2, l2);
  const uint64_t l = l1 + l2;
  return redc(h1 + h2 + (l < l1 ? 1 : 0), l, q, qinv);
}

// Products of two variables, two of mul_tw's Montgomery steps, so that they come
// out off by 2^-60 (cancelled elsewhere: folded into the N^-1 scaling of the
// inverse transform that follows, or into the key switch's last product).  With a
// split at bit 30 (a below 2^62) and b1 four times the high word of b (below 2^62
// too), a b = a b0 + 2^30 a b1: the first step divides a b0 by 2^30, the second
// its result U plus a b1.  U enters the second step's p0 whole, so
// U + a0 b1 + m qlo has to stay below 2^64, with U < a b0 / 2^30 + 4q, m qlo < 2^62
// and results below a b1 / 2^30 + 4.1q:
//   34..55 bits  a, b < 3q: U < 16q < 2^59 (the sum of two products 28q), results
//                below 5q (the sum 6q);
//   56..60 bits  a < q, b < 2q: U < 8q < 2^63, a0 b1 < 2^61, results below 7q;
//   33 or fewer  lazy words (below 207q < 2^41): results below 5q.
//
// 12 instructions a product and 16 the sum of two, with the splits shared between
// the products of a ciphertext tensor 46 in all; Montgomery products of whole
// 64-bit words (R = 2^64) took 117 as compiled, 51 of them moves that zero-extend
// 32-bit halves.
struct Split30 { uint32_t lo, hi; };
__device__ __forceinline__ Split30 split30(uint64_t a) {
  return Split30{lo32(a) & ((1u << 30) - 1), (uint32_t)(a >> 30)};
}
__device__ __forceinline__ uint64_t redc30(uint64_t p0, uint64_t p1, const NttConst &c, uint32_t four) {
  const uint32_t m = lo32(p0) * c.qi;
  p0 = mad32(m, c.qlo, p0);
  p1 = mad32(m, c.qhi, p1);
  return mad32(hi32(p0), four, p1);
}
// x + a b 2^-60 mod q
__device__ __forceinline__ uint64_t mont30_mul_add(Split30 a, uint64_t b, uint64_t x, const NttConst &c,
                                                   uint32_t four) {
  const uint32_t b0 = lo32(b), b1 = hi32(b) << 2;
  const uint64_t u = redc30(mad32(a.lo, b0, 0), mad32(a.hi, b0, 0), c, four);
  return redc30(mad32(a.lo, b1, u), mad32(a.hi, b1, x), c, four);
}
__device__ __forceinline__ uint64_t mont30_mul(Split30 a, uint64_t b, const NttConst &c, uint32_t four) {
  return mont30_mul_add(a, b, 0, c, four);
}
// (a b + d e) 2^-60 mod q
__device__ __forceinline__ uint64_t mont30_mad(Split30 a, uint64_t b, Split30 d, uint64_t e, const NttConst &c,
                                               uint32_t four) {
  const uint32_t b0 = lo32(b), b1 = hi32(b) << 2, e0 = lo32(e), e1 = hi32(e) << 2;
  const uint64_t u = redc30(mad32(d.lo, e0, mad32(a.lo, b0, 0)), mad32(d.hi, e0, mad32(a.hi, b0, 0)), c, four);
  return redc30(mad32(d.lo, e1, mad32(a.lo, b1, u)), mad32(d.hi, e1, mad32(a.hi, b1, 0)), c, four);
}

}  // namespace hentt
