// The lazy bounds of every transform schedule, followed stage by stage: the
// geometry, the corrections and the offsets are the kernels' own (schedule.hpp,
// host_tables.hpp); the words are held as upper bounds, for the largest modulus of
// each bit length.  A product by a root power takes any 64-bit word and leaves less
// than 12q; est3 takes any 64-bit word and leaves less than 3q (moduli of 34 bits and
// more; smaller ones pass); reduce_word takes 64 bits (k >= 34) or k + 21 bits.
#include <stdint.h>
#include <stdio.h>
#include <algorithm>
#include <vector>
#define HENTT_HOST_TEST 1
#include "../paper_2109_14704_amd/csrc/host_tables.hpp"
#include "../paper_2109_14704_amd/csrc/schedule.hpp"

typedef unsigned __int128 u128;
using namespace hentt;

static long fails = 0, checks = 0;
#define EXPECT(c, ...)                       \
  do {                                       \
    ++checks;                                \
    if (!(c)) {                              \
      if (fails++ < 20) printf(__VA_ARGS__); \
    }                                        \
  } while (0)
static const u128 TOP = (u128)1 << 64;

struct Mod {
  int k;
  u128 q;      // the largest of k bits
  bool fix() const { return !uncorrected((uint32_t)k); }
  u128 est3(u128 x) const { return k >= 34 ? std::min(x, 3 * q) : x; }
  u128 reducible() const { return k >= 34 ? TOP : (u128)1 << (k + 21); }
};

// All bounds below are exclusive.  Forward: X' and Y' below X + 12q.
static u128 fwd_stages(const Mod &m, u128 x, int stages) {
  for (int s = 0; s < stages; ++s) {
    EXPECT(x <= TOP, "forward input, k=%d stage %d\n", m.k, s);
    x = (m.fix() ? m.est3(x) : x) + 12 * m.q;
    EXPECT(x <= TOP, "forward output, k=%d stage %d\n", m.k, s);
  }
  return x;
}

// One inverse round at stages LO .. LO + R - 1 of 2^logn, all words entering below
// `in`; returns the largest word it leaves.
template <int R, int LBIN, int LBOUT> u128 inv_round(const Mod &m, u128 in, int LO, int logn) {
  const bool fix = m.fix();
  std::vector<u128> x(1u << R, in);
  if (!fix) EXPECT(in <= m.q << LBIN, "entry, k=%d R=%d LBIN=%d\n", m.k, R, LBIN);
  if (fix && m.k >= 34) EXPECT(in <= 8 * m.q, "entry, k=%d R=%d\n", m.k, R);
  for (int u = 0; u < R; ++u) {
    const int v = LO + u, d = 1 << u;
    const u128 off = m.q << inv_off_log((uint32_t)m.k, fix, LBIN, u, v);
    const bool last = v == logn - 1;
    for (int i = 0; i < (1 << R); ++i) {
      if (i & d) continue;
      const u128 X = x[i], Y = x[i + d];
      EXPECT(Y <= off + 1, "offset, k=%d R=%d u=%d v=%d\n", m.k, R, u, v);
      EXPECT(X + off <= TOP && X + Y <= TOP, "overflow, k=%d R=%d u=%d v=%d\n", m.k, R, u, v);
      x[i] = last ? 12 * m.q : X + Y;
      x[i + d] = 12 * m.q;
    }
    if (last) continue;
    for (int i = 0; i < (1 << R); ++i)
      if (fix ? inv_fix(R, u, i & d) : u == R - 1 && inv_over<R, LBIN, LBOUT>(i)) x[i] = m.est3(x[i]);
  }
  u128 out = 0;
  const bool end = LO + R == logn;
  for (u128 w : x) {
    out = std::max(out, w);
    if (!end && !fix) EXPECT(w <= m.q << LBOUT, "exit, k=%d R=%d LBIN=%d LBOUT=%d\n", m.k, R, LBIN, LBOUT);
    if (!end && fix && m.k >= 34) EXPECT(w <= 4 * m.q, "exit, k=%d R=%d\n", m.k, R);
  }
  if (end) EXPECT(out <= m.reducible(), "final reduction, k=%d\n", m.k);
  return out;
}

// inv_block_rounds: rounds over stages [LO, ST) of 2^LOGN.
template <int LOGN, int ST, int E, int LO = 0, int R = (ST < E ? ST : E)> u128 inv_block(const Mod &m, u128 in) {
  const u128 out = inv_round<R, LB_ROUND, (LO + R < ST ? LB_ROUND : LB_PASS)>(m, in, LO, LOGN);
  if constexpr (LO + R < ST) {
    constexpr int LO2 = LO + R, R2 = (ST - LO2) < E ? (ST - LO2) : E;
    return inv_block<LOGN, ST, E, LO2, R2>(m, out);
  } else {
    return out;
  }
}
// The inverse column pass: EC >= 6 through LDS in two rounds, else one round.
template <int LOGN, int EC> void inv_cols(const Mod &m, u128 in) {
  if constexpr (EC >= 6) {
    const u128 mid = inv_round<EC - 4, LB_PASS, LB_ROUND>(m, in, LOGN - EC, LOGN);
    inv_round<4, LB_ROUND, LB_PASS>(m, mid, LOGN - 4, LOGN);
  } else {
    inv_round<EC, LB_PASS, LB_PASS>(m, in, LOGN - EC, LOGN);
  }
}
template <int LOGN, int EC, int E> void inverse(const Mod &m) {
  // canonical words and products of variables (below 7q, 2q outside the key switch)
  for (u128 in : {m.q, 7 * m.q}) {
    if (in > m.q && m.fix() && m.k >= 34) in = 2 * m.q;   // 56 bits and more: 64-bit Montgomery products
    const u128 mid = inv_block<LOGN, LOGN - EC, E>(m, in);
    if constexpr (EC > 0) inv_cols<LOGN, EC>(m, mid);
    else (void)mid;
  }
}
template <int LOGN> void whole(const Mod &m) { inverse<LOGN, 0, whole_e(LOGN)>(m); }
template <int LOGN> void two_pass(const Mod &m) { inverse<LOGN, two_pass_cols(LOGN), 3>(m); }

int main() {
  for (int k = 8; k <= 60; ++k) {
    const Mod m{k, ((u128)1 << k) - 1};
    const uint64_t q = (uint64_t)m.q;
    // forward: canonical words; the rescale's and the key switch's lifted words, at every N
    for (int logn = 6; logn <= 17; ++logn) {
      for (u128 in : {m.q, k < 34 ? 3 * m.q : ((u128)1 << 60) + m.q, k < 34 ? 2 * m.q : (u128)1 << 60}) {
        const u128 t = fwd_stages(m, in, logn);
        EXPECT(t <= m.reducible(), "forward reduction, k=%d logn=%d\n", k, logn);
        const u128 off = host::rs_off(q);
        EXPECT(t <= off + 1 && m.q + off <= TOP && off % m.q == 0, "rescale offset, k=%d logn=%d\n", k, logn);
        if (k < 34) EXPECT(2 * t * t <= (m.q << 64), "Montgomery products of small moduli, k=%d logn=%d\n", k, logn);
      }
    }
    // inverse: the default schedules and the tuner's
    whole<6>(m), whole<7>(m), whole<8>(m), whole<9>(m), whole<10>(m), whole<11>(m), whole<12>(m), whole<13>(m), whole<14>(m);
    inverse<9, 0, 3>(m), inverse<14, 2, 3>(m), inverse<15, 5, 3>(m), inverse<17, 5, 3>(m), inverse<16, 6, 4>(m);
    two_pass<13>(m), two_pass<14>(m), two_pass<15>(m), two_pass<16>(m), two_pass<17>(m);
    inverse<13, 7, 2>(m), inverse<14, 7, 2>(m), inverse<15, 7, 3>(m), inverse<16, 8, 3>(m), inverse<16, 8, 2>(m),
        inverse<17, 7, 3>(m);
    // the persistent batch: blocks of 2^12 with 16 words per lane, 1 to 5 column stages
    inverse<12, 0, 4>(m), inverse<13, 1, 4>(m), inverse<14, 2, 4>(m), inverse<15, 3, 4>(m), inverse<16, 4, 4>(m),
        inverse<17, 5, 4>(m);
  }
  printf(fails ? "FAIL %ld of %ld\n" : "OK %ld %ld\n", fails, checks);
  return fails ? 1 : 0;
}
