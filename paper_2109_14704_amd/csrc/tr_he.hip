// Dispatch of the homomorphic routines built on the transforms: rescale (RS),
// relinearization with the RNS digit key switch (Relin) and the encrypted
// element-wise polynomial matrix product.
#include <algorithm>

#include "host_tables.hpp"
#include "keyswitch_kernels.hpp"
#include "matmul_kernels.hpp"
#include "rescale_kernels.hpp"
#include "runtime.hpp"

namespace hentt_rt {
namespace {

// ---------------------------------------------------------------- rescale
// Constants of RS from a level of `level` limbs to level - 1 (section II-A):
// per remaining limb i, floor(2^64 / q_i), q_i - (h mod q_i) with
// h = (qL - 1) / 2, and qL^-1 mod q_i as a root power.  Made once per
// (tables, level) with a synchronous upload, like the tables themselves.
int rs_constants(Storage *s, uint32_t level, const RsLimb **out) {
  std::lock_guard<std::mutex> lk(s->rs_mu);
  auto it = s->rs.find(level);
  if (it != s->rs.end()) {
    *out = it->second;
    return HENTT_OK;
  }
  const uint32_t L = level - 1;
  const uint64_t qL = s->moduli[L], h = (qL - 1) / 2;
  std::vector<RsLimb> host(L);
  for (uint32_t i = 0; i < L; ++i) {
    const uint64_t q = s->moduli[i];
    host[i].mu = (uint64_t)(((host::u128)1 << 64) / q);
    host[i].nh = q - h % q;
    host[i].w = host::tw_m(host::pow(qL % q, q - 2, q), q);
    host[i].off = host::rs_off(q);
  }
  RsLimb *d = nullptr;
  hipError_t e = hipMalloc(&d, L * sizeof(RsLimb));
  if (e == hipSuccess) e = hipMemcpy(d, host.data(), L * sizeof(RsLimb), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    if (d) (void)hipFree(d);
    return hip_fail(e);
  }
  s->rs[level] = d;
  *out = d;
  return HENTT_OK;
}

// Stage split of the rescale's forward transforms: whole up to 2^13, the two-pass
// split above (2^16, 64 polynomials of 24 limbs, when measured: 753 us with seven column
// stages, 771 with six, 762 with five in registers; 734 since).
template <int LOGN> struct RsPlan {
  static constexpr bool WHOLE = LOGN <= 13;
  static constexpr int EC = two_pass_cols(LOGN), E = 3, ST = LOGN - EC, B = block_words(ST, E);
};

// Block pass of the inverse transform of `limbs` limbs from limb `first` on, read
// where they lie (limb l of entry b at src + b src_sb + l N) into dst; the column
// passes of the rescale and the key switch take the rest.
template <int LOGN>
void inv_blocks_from(const Storage *s, uint32_t first, uint32_t limbs, const uint64_t *src, uint64_t src_sb,
                    uint64_t *dst, uint32_t batch, hipStream_t st) {
  constexpr int E = 3, ST = LOGN - two_pass_cols(LOGN), B = block_words(ST, E);
  const uint64_t sb = (uint64_t)limbs << LOGN;
  const InvIO io{src, dst, src_sb, sb};
  LaunchTimer lt_("k_inv_blocks", LOGN, st);
  hipLaunchKernelGGL((k_inv_blocks<LOGN, ST, B, E>), dim3((batch * limbs) << (LOGN - B)), dim3(1 << (B - E)), 0, st, io,
                     s->d_twm + (size_t)first * 2 * (1u << LOGN), s->d_nc + first, batch, limbs);
}

// The last limb of every batch entry goes through `last`, [batch][N] words of the
// library's own: inverse-transformed modulo qL, read where it lies.  Two-pass
// sizes leave its column pass to k_rs_cols while that launch fits the chip at once
// (kRsWaves, four waves per SIMD): N = 2^15, 8 limbs, 2 polynomials, 16.5 us for
// the two column passes, 12 for the one; at 64 polynomials 40 to 47 and 57.
constexpr uint64_t kRsWaves = 4096;
template <int LOGN> int launch_rescale_ntt(RsArgs a, Storage *s, uint64_t *last, hipStream_t st) {
  const uint32_t units = a.batch * a.L;
  const uint64_t *cl = a.c + ((uint64_t)a.L << LOGN), sb = (uint64_t)(a.L + 1) << LOGN;
  using P = RsPlan<LOGN>;
  a.tl = last;
  Storage one;  // limb L's tables alone (a view: owns nothing)
  one.log_n = LOGN;
  one.limbs = 1;
  one.d_twm = s->d_twm + ((size_t)a.L * 2 << LOGN);
  one.d_nc = s->d_nc + a.L;
  one.d_mont = s->d_mont + a.L;
  one.device = s->device;
  const hentt_tables lv{&one, 1};
  if constexpr (P::WHOLE) {
    const int rc = run_inverse_from(&lv, cl, sb, last, a.batch, st);
    if (rc) return rc;
    LaunchTimer lt_("k_rs_whole", LOGN, st);
    hipLaunchKernelGGL((k_rs_whole<LOGN, whole_e(LOGN)>), dim3(units), dim3(1 << (LOGN - whole_e(LOGN))), 0, st, a, s->d_twm, s->d_nc);
  } else {
    constexpr uint32_t tiles = cols_blocks_per_unit<LOGN, P::EC>(), lanes = cols_lanes<P::EC>();
    const dim3 g(units * tiles), blk(lanes);
    if ((uint64_t)units * tiles * (lanes / 64) <= kRsWaves) {
      inv_blocks_from<LOGN>(s, a.L, 1, cl, sb, last, a.batch, st);
      LaunchTimer lt_("k_rs_cols", LOGN, st);
      hipLaunchKernelGGL((k_rs_cols<LOGN, P::EC, true>), g, blk, 0, st, a, s->d_twm, s->d_nc);
    } else {
      const int rc = run_inverse_from(&lv, cl, sb, last, a.batch, st);
      if (rc) return rc;
      LaunchTimer lt_("k_rs_cols", LOGN, st);
      hipLaunchKernelGGL((k_rs_cols<LOGN, P::EC, false>), g, blk, 0, st, a, s->d_twm, s->d_nc);
    }
    LaunchTimer lt_("k_rs_blocks", LOGN, st);
    hipLaunchKernelGGL((k_rs_blocks<LOGN, P::ST, P::B, P::E>), dim3(units << (LOGN - P::B)), dim3(1 << (P::B - P::E)), 0, st, a,
                       s->d_twm, s->d_nc);
  }
  HIPCHK(hipGetLastError());
  return HENTT_OK;
}
typedef int (*rs_fn)(RsArgs, Storage *, uint64_t *, hipStream_t);
#define RS_ENTRY(n) launch_rescale_ntt<n>,
const rs_fn k_rs_table[] = {HENTT_SIZES(RS_ENTRY)};

// ------------------------------------------------------- relinearization
// Key-switching constants of the level with L1 limbs (the last one is P).
int ks_consts(Storage *s, uint32_t L1, const KsLimb **out) {
  std::lock_guard<std::mutex> lk(s->rs_mu);
  auto it = s->ks.find(L1);
  if (it != s->ks.end()) {
    *out = it->second;
    return HENTT_OK;
  }
  const uint64_t P = s->moduli[L1 - 1];
  std::vector<KsLimb> kc(L1);
  for (uint32_t t = 0; t < L1; ++t) {
    const uint64_t q = s->moduli[t];
    kc[t].mu = (uint64_t)(((host::u128)1 << 64) / q);
    kc[t].r = host::tw_m((1ull << 60) % q, q);
    kc[t].pm = host::tw_m(P % q, q);
  }
  KsLimb *d = nullptr;
  hipError_t e = hipMalloc(&d, L1 * sizeof(KsLimb));
  if (e == hipSuccess) e = hipMemcpy(d, kc.data(), L1 * sizeof(KsLimb), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    if (d) (void)hipFree(d);
    return hip_fail(e);
  }
  s->ks[L1] = d;
  *out = d;
  return HENTT_OK;
}

// Key-switch split: the digit loop holds two accumulator arrays, so whole
// transforms only up to 2^12 (512 lanes); above, the two-pass split (2^15, 32
// ciphertexts, 8 primes, the key switch alone when measured: 546 us with six column
// stages, 549 with seven, 595 with five in registers; 455 since).
template <int LOGN> struct KsPlan {
  static constexpr bool WHOLE = LOGN <= 12;
  static constexpr int EC = two_pass_cols(LOGN);
  static constexpr int E = 3, ST = LOGN - EC, B = block_words(ST, E);  // words per lane in the block kernel (3: occupancy over radix)
};

// Blocks of a small batch spread their digits over workgroups up to this many
// waves in all (N = 2^15: 77 -> 69 us at 8 primes and one entry, 95 -> 90 at two
// entries, no difference at three; 86 -> 68 us at 2^14, 12 primes, one entry).
constexpr uint32_t kKsWaves = 2304;

// Workgroups a digit's column tile spreads its target primes over: each repeats
// the tile's inverse stages, so no more than fill kColWaves waves (2^15, 8 primes,
// 32 and 4 entries: 600 and 117 us with 4096, 612 and 123 with 8192, 620 and 122
// with 16384; 2048 differs by the run).
constexpr uint32_t kColWaves = 4096;
template <int EC> uint32_t col_splits(uint64_t groups, uint32_t primes) {
  const uint64_t waves = groups * (cols_lanes<EC>() / 64);
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(primes, kColWaves / waves));
}

// d: [batch][l][N] words of the library's own for the digits, c2 in the
// coefficient domain modulo its own primes (two-pass sizes: up to the column pass).
template <int LOGN> int launch_keyswitch(KsArgs a, Storage *s, uint64_t *d, hipStream_t st) {
  const uint32_t L1 = a.l + 1;
  const uint64_t P2 = (uint64_t)a.l << LOGN;
  using P = KsPlan<LOGN>;
  a.d = d;
  if constexpr (P::WHOLE) {
    const hentt_tables lv{s, a.l};
    const int rc = run_inverse_from(&lv, a.c + 2 * P2, 3 * P2, d, a.batch, st);
    if (rc) return rc;
    LaunchTimer lt_("k_ks_whole", LOGN, st);
    hipLaunchKernelGGL((k_ks_whole<LOGN, whole_e(LOGN)>), dim3(a.batch * L1), dim3(1 << (LOGN - whole_e(LOGN))), 0, st, a, s->d_twm, s->d_nc);
  } else {
    inv_blocks_from<LOGN>(s, 0, a.l, a.c + 2 * P2, 3 * P2, d, a.batch, st);
    constexpr uint32_t tiles = cols_blocks_per_unit<LOGN, P::EC>();
    a.col_splits = col_splits<P::EC>((uint64_t)a.batch * a.l * tiles, L1);
    {
      LaunchTimer lt_("k_ks_cols", LOGN, st);
      hipLaunchKernelGGL((k_ks_cols<LOGN, P::EC>), dim3(a.batch * a.l * a.col_splits * tiles),
                         dim3(cols_lanes<P::EC>()), 0, st, a, s->d_twm, s->d_nc);
    }
    {
      LaunchTimer lt_("k_ks_blocks", LOGN, st);
      hipLaunchKernelGGL((k_ks_blocks<LOGN, P::ST, P::B, P::E>), dim3((a.splits * a.batch * L1) << (LOGN - P::B)),
                         dim3(1 << (P::B - P::E)), 0, st, a, s->d_twm, s->d_nc);
    }
    if (a.splits > 1) {
      LaunchTimer lt_("k_ks_sum", LOGN, st);
      hipLaunchKernelGGL((k_ks_sum<LOGN>), dim3(a.batch * 2 * L1 << (LOGN - 8)), dim3(256), 0, st, a, s->d_nc);
    }
  }
  HIPCHK(hipGetLastError());
  return HENTT_OK;
}
typedef int (*ks_fn)(KsArgs, Storage *, uint64_t *, hipStream_t);
#define KS_ENTRY(n) launch_keyswitch<n>,
const ks_fn k_ks_table[] = {HENTT_SIZES(KS_ENTRY)};

}  // namespace

int run_rescale(const hentt_tables *t, const uint64_t *c, uint64_t *out, uint32_t batch, bool ntt, hipStream_t st) {
  Storage *s = t->s;
  const uint32_t ln = s->log_n, level = t->limbs, L = level - 1;
  const uint64_t N = 1ull << ln;
  const RsLimb *rs = nullptr;
  int rc = rs_constants(s, level, &rs);
  if (rc) return rc;
  RsArgs a{};
  a.c = c;
  a.out = out;
  a.rs = rs;
  a.qL = s->moduli[L];
  a.h = (a.qL - 1) / 2;
  a.batch = batch;
  a.L = L;
  if (!ntt) {
    const uint32_t tiles = (uint32_t)((N + 2047) / 2048);
    LaunchTimer lt_("k_rs_coeff", (int)ln, st);
    hipLaunchKernelGGL(k_rs_coeff, dim3(batch * L * tiles), dim3(256), 0, st, a, s->d_nc, ln, tiles);
    HIPCHK(hipGetLastError());
    return HENTT_OK;
  }
  const uint32_t piece = batch_piece(ln, L, batch);
  void *tl = nullptr;
  rc = pool_get((size_t)piece * N * 8, st, &tl);
  if (rc) return rc;
  for (uint64_t b = 0; b < batch && !rc; b += piece) {
    a.c = c + (b * level << ln);
    a.out = out + (b * L << ln);
    a.batch = (uint32_t)std::min<uint64_t>(piece, batch - b);
    rc = k_rs_table[ln - HENTT_LOG_N_MIN](a, s, (uint64_t *)tl, st);
  }
  pool_put(tl);
  return rc;
}

int run_relin(const hentt_tables *t, const uint64_t *c, const uint64_t *ksk, uint64_t *out, uint32_t batch,
              hipStream_t st) {
  Storage *s = t->s;
  const uint32_t ln = s->log_n, L1 = t->limbs, l = L1 - 1;
  const uint64_t N = 1ull << ln, P = (uint64_t)l * N;
  const KsLimb *kc = nullptr;
  int rc = ks_consts(s, L1, &kc);
  if (rc) return rc;
  const bool two_pass = ln > 12;  // KsPlan<>::WHOLE
  const size_t d_bytes = (size_t)batch * P * 8, acc_bytes = (size_t)batch * 2 * L1 * N * 8;
  const size_t e_bytes = two_pass ? (size_t)batch * l * L1 * N * 8 : 0;
  const uint64_t waves = (uint64_t)batch * L1 * N >> 9;
  uint32_t splits = two_pass ? (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(l / 2, kKsWaves / waves)) : 1;
  // The partial sums only make the call faster: where the pool cannot grow for them
  // (memory, or a capture, which an allocation would end), it does without.
  void *buf = nullptr;
  rc = pool_get(d_bytes + acc_bytes + e_bytes + (splits > 1 ? splits * acc_bytes : 0), st, &buf,
                splits == 1 || !capturing(st));
  if (rc == HENTT_ENOMEM && splits > 1) {
    splits = 1;
    rc = pool_get(d_bytes + acc_bytes + e_bytes, st, &buf);
  }
  if (rc) return rc;
  uint64_t *d = (uint64_t *)buf, *acc = d + batch * P, *e = acc + (size_t)batch * 2 * L1 * N, *part = e + e_bytes / 8;
  KsArgs a{};
  a.ksk = ksk;
  a.e = two_pass ? e : nullptr;
  a.acc = acc;
  a.c = c;
  a.kc = kc;
  a.part = splits > 1 ? part : nullptr;
  a.splits = splits;
  a.batch = batch;
  a.l = l;
  rc = k_ks_table[ln - HENTT_LOG_N_MIN](a, s, d, st);
  // divide by P with rounding, over q_0 .. q_{l-1}: [batch][2][l+1] -> [batch][2][l];
  // the accumulators already hold P c_s, so this yields (c0, c1) + round(P^-1 c2 evk)
  if (!rc) rc = run_rescale(t, acc, out, batch * 2, true, st);
  pool_put(buf);
  return rc;
}

// ------------------------------------------------------------ matMul
int run_matmul(const hentt_tables *t, const uint64_t *A, const uint64_t *B, uint64_t *C, uint32_t m, uint32_t n,
               uint32_t k, hipStream_t st) {
  const uint32_t ln = t->s->log_n, L = t->limbs;
  const uint64_t P = (uint64_t)L << ln;
  if ((uint64_t)m * n * L * (((1ull << ln) + 2047) >> 11) > 0x7fffffffu) return HENTT_EINVAL;  // as the header states
  const uint32_t tiles = ln > 8 ? 1u << (ln - 8) : 1u;
  // Runs of up to CT_J columns; shorter ones where that leaves the chip short of two
  // workgroups per CU, since a workgroup's time is its chain of k steps over its run
  // (4 limbs, 10 x 9 x 8: N = 2^8 11.1 us with runs of 5 columns, 8.4 with single ones,
  // 2^10 16.4 and 14.6, no difference from 2^11 on).
  const uint64_t per_run = (uint64_t)L * tiles * m, want = 2ull * t->s->cus;
  const uint32_t runs =
      (uint32_t)std::min<uint64_t>(n, std::max<uint64_t>((n + CT_J - 1) / CT_J, (want + per_run - 1) / per_run));
  const uint64_t groups = (uint64_t)L * runs * tiles, per_row = (groups + 7) / 8 * 8;
  if (per_row > kMaxItems / 256) return HENTT_EINVAL;
  const uint32_t rows = (uint32_t)std::min<uint64_t>(m, kMaxItems / 256 / per_row);
  for (uint64_t i = 0; i < m; i += rows) {
    const uint32_t mi = (uint32_t)std::min<uint64_t>(rows, m - i);
    const MatmulArgs p{A + i * k * 2 * P, B, C + i * n * 3 * P, mi, n, k, L, ln, tiles, runs, (uint32_t)groups};
    LaunchTimer lt_("k_ct_matmul", (int)ln, st);
    hipLaunchKernelGGL(k_ct_matmul, dim3((uint32_t)(per_row * mi)), dim3(256), 0, st, p, t->s->d_nc, t->s->d_mat);
  }
  HIPCHK(hipGetLastError());
  return HENTT_OK;
}

}  // namespace hentt_rt
