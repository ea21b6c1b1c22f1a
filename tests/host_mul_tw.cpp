// CPU property test of the transforms' arithmetic (modarith.hpp and
// host_tables.hpp built for the host): products by a root power in split
// Montgomery form, the butterflies built on them, the quotient estimates and
// the canonical reduction, against exact 128-bit arithmetic at the edges of
// their ranges, and the lazy bounds of whole transforms followed stage by stage.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <random>
#define HENTT_HOST_TEST 1
#include "../paper_2109_14704_amd/csrc/host_tables.hpp"
#include "../paper_2109_14704_amd/csrc/modarith.hpp"

typedef unsigned __int128 u128;
using namespace hentt;

static int fails = 0;
#define EXPECT(c, ...)                       \
  do {                                       \
    if (!(c)) {                              \
      if (fails++ < 10) printf(__VA_ARGS__); \
    }                                        \
  } while (0)

static uint64_t mm(uint64_t a, uint64_t b, uint64_t q) { return (uint64_t)((u128)a * b % q); }

// Constants of any odd q of k bits (the arithmetic does not need a prime).
static NttConst consts(uint64_t q, int k) {
  LimbConst c{};
  c.m.q = q;
  c.k = (uint32_t)k;
  c.mu = (uint64_t)(((u128)1 << (2 * k)) / q);
  c.ninv = q - 1;
  c.ninvw = 1;
  return host::ntt_const(c);
}

int main(int argc, char **argv) {
  const long iters = argc > 1 ? atol(argv[1]) : 200000;
  std::mt19937_64 g(30);
  for (long it = 0; it < iters; ++it) {
    const int k = 8 + (int)(it % 53);  // bit length 8..60
    uint64_t q = ((g() >> (64 - k)) | (1ull << (k - 1))) | 1;
    if (it % 7 == 0) q = (1ull << k) - 1;
    if (it % 11 == 0) q = (1ull << (k - 1)) + 1;
    const NttConst c = consts(q, k);
    const uint64_t W = it % 5 == 0 ? q - 1 : g() % q;
    const TwM w = host::tw_m(W, q);
    const uint64_t ys[4] = {g(), ~0ull, 0xffffffffull, 0xffffffff00000000ull};
    for (uint64_t y : ys) {
      const uint64_t t = mul_tw(w, y, c, 4);
      EXPECT((u128)t < (u128)12 * q && t % q == mm(W, y % q, q), "mul_tw q=%llx\n", (unsigned long long)q);
      const uint64_t x = g() % (4 * q), s = mul_tw_add(w, y, x, c, 4);
      EXPECT(s - x == t, "mul_tw_add\n");
      uint64_t X = x, Y = y;
      ct_bfly_m(X, Y, w, c, 4);
      EXPECT(X == x + t && Y == x + 12 * q - t, "ct_bfly_m q=%llx\n", (unsigned long long)q);
      const uint64_t b = 8 * q, a = g() % b, d = it % 3 ? g() % b : b - 1;
      uint64_t A = a, D = d;
      gs_bfly_m(A, D, w, b, c, 4);
      EXPECT(A == a + d && (u128)D < (u128)12 * q && D % q == mm(W, (a % q + q - d % q) % q, q), "gs_bfly_m\n");
      {  // products of two variables, at the bounds of each size's factors
        const uint64_t qa = k < 34 ? 207 * q : k <= 55 ? 3 * q : q, qb = k < 34 ? 207 * q : k <= 55 ? 3 * q : 2 * q;
        const uint64_t a0 = it % 4 ? g() % qa : qa - 1, a1 = it % 6 ? g() % qa : qa - 1;
        const uint64_t b0 = it % 3 ? g() % qb : qb - 1, b1 = it % 2 ? g() % qb : qb - 1;
        const uint64_t r60 = (1ull << 60) % q, b = (k <= 55 ? 5 : 7) * q;
        const uint64_t p = mont30_mul(split30(a0), b0, c, 4), s2 = mont30_mul_add(split30(a1), b1, 3 * q, c, 4);
        EXPECT(p < b && s2 < b + 3 * q, "mont30 ranges q=%llx\n", (unsigned long long)q);
        EXPECT(mm(p % q, r60, q) == mm(a0 % q, b0 % q, q), "mont30_mul q=%llx\n", (unsigned long long)q);
        EXPECT(mm(s2 % q, r60, q) == mm(a1 % q, b1 % q, q), "mont30_mul_add q=%llx\n", (unsigned long long)q);
        if (k <= 55) {
          const uint64_t ps = mont30_mad(split30(a0), b0, split30(a1), b1, c, 4);
          EXPECT(ps < 6 * q, "mont30_mad range q=%llx\n", (unsigned long long)q);
          EXPECT(mm(ps % q, r60, q) == (mm(a0 % q, b0 % q, q) + mm(a1 % q, b1 % q, q)) % q, "mont30_mad\n");
        }
      }
      if (k >= 34) {
        const uint64_t e = est3(y, c);
        EXPECT((u128)e < (u128)3 * q && e % q == y % q, "est3 q=%llx\n", (unsigned long long)q);
        EXPECT(reduce_word(y, c) == y % q, "reduce_word q=%llx\n", (unsigned long long)q);
      } else {
        EXPECT(est3(y, c) == y, "est3 of a small modulus\n");
        const uint64_t top = (1ull << (k + 21)) - 1;
        const uint64_t xs[5] = {y & top, top, 0, q * (top / q), q * (top / q) - 1};
        for (uint64_t v : xs) EXPECT(reduce_word(v, c) == v % q, "reduce_word small q=%llx\n", (unsigned long long)q);
      }
    }
  }
  // Lazy bounds, in units of q, of 17 stages: forward without corrections up to
  // 56 bits (from 3q) and corrected every stage above; inverse words of any
  // modulus up to 33 bits at 16q 2^v.
  EXPECT(3 + 12 * 17 < 256, "forward bound\n");
  EXPECT(3 + 12 < 16, "corrected forward bound\n");
  EXPECT(33 + 4 + 17 <= 54 && 33 + 21 <= 54, "small inverse bound\n");
  printf(fails ? "FAIL %d\n" : "OK\n", fails);
  return fails ? 1 : 0;
}
