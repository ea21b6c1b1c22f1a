// Dispatch of the plain batched transforms (hentt_ntt_fwd / hentt_ntt_inv)
// and of the kernel-instance choices the autotuner selects between.
//
// Every N has a list of compiled instances ("candidates"): a whole transform
// per workgroup (one HBM round trip), or a column pass of EC stages followed
// by blocks of 2^(log_n - EC) words with 2^E words per lane.  Candidate 0 is
// the default; the autotuner may select another per (operation, N, shape
// class), where the shape class groups the number of (batch entry, limb)
// units of a call.
#include <algorithm>

#include "runtime.hpp"

namespace hentt_rt {
namespace {

// Whole transform of one (batch entry, limb) per workgroup.
template <int LOGN, int E>
void launch_fwd_whole(const hentt_tables *t, uint64_t *x, uint32_t batch, hipStream_t st) {
  LaunchTimer lt_("k_fwd_whole", LOGN, st);
  hipLaunchKernelGGL((k_fwd_whole<LOGN, E>), dim3(batch * t->limbs), dim3(1 << (LOGN - E)), 0, st, x, t->s->d_twm,
                     t->s->d_nc, batch, t->limbs);
}
template <int LOGN>
void launch_whole(const hentt_tables *t, const InvIO &io, uint32_t batch, bool inv, hipStream_t st) {
  constexpr int E = whole_e(LOGN);
  const uint32_t L = t->limbs, units = batch * L;
  if (inv) {
    LaunchTimer lt_("k_inv_whole", LOGN, st);
    hipLaunchKernelGGL((k_inv_whole<LOGN, E>), dim3(units), dim3(1 << (LOGN - E)), 0, st, io, t->s->d_twm, t->s->d_nc,
                       batch, L);
    return;
  }
  if constexpr (LOGN == 13) {
    // The 16 waves of a forward 2^13 with 8 words per lane (78 VGPRs) have a CU to
    // themselves and stand at its barriers together.  With 16 words and 128 VGPRs two
    // workgroups share the CU: slower while there are no two (256 units 13.9 and 14.8
    // us), even at 512, faster from there on (1024 units 50.1 and 46.4, 4096 187 and 176;
    // with 60-bit moduli 54.6 and 50.9, 197 and 188).
    if (units > 2u * t->s->cus) {
      launch_fwd_whole<LOGN, 4>(t, io.dst, batch, st);
      return;
    }
  }
  launch_fwd_whole<LOGN, E>(t, io.dst, batch, st);
}

// Column pass of EC stages and block pass on 2^(LOGN - EC) words, 2^E per lane.
template <int LOGN, int EC, int E>
void launch_two_pass(const hentt_tables *t, const InvIO &io, uint32_t batch, bool inv, hipStream_t st) {
  constexpr int ST = LOGN - EC, B = block_words(ST, E);
  const TwM *tw = t->s->d_twm;
  const NttConst *lc = t->s->d_nc;
  const uint32_t L = t->limbs, units = batch * L;
  const dim3 gcols(units * cols_blocks_per_unit<LOGN, EC>());
  if (!inv) {
    {
      LaunchTimer lt_("k_cols_fwd", LOGN, st);
      hipLaunchKernelGGL((k_cols<LOGN, EC, false>), gcols, dim3(cols_lanes<EC>()), 0, st, col_args(io.dst, io.dst_sb), tw, lc,
                         batch, L);
    }
    LaunchTimer lt_("k_fwd_blocks", LOGN, st);
    hipLaunchKernelGGL((k_fwd_blocks<LOGN, ST, B, E>), dim3(units << (LOGN - B)), dim3(1 << (B - E)), 0, st, io.dst, tw, lc,
                       batch, L);
  } else {
    {
      LaunchTimer lt_("k_inv_blocks", LOGN, st);
      hipLaunchKernelGGL((k_inv_blocks<LOGN, ST, B, E>), dim3(units << (LOGN - B)), dim3(1 << (B - E)), 0, st, io, tw, lc,
                         batch, L);
    }
    LaunchTimer lt_("k_cols_inv", LOGN, st);
    hipLaunchKernelGGL((k_cols<LOGN, EC, true>), gcols, dim3(cols_lanes<EC>()), 0, st, col_args(io.dst, io.dst_sb), tw, lc,
                       batch, L);
  }
}

typedef void (*tr_fn)(const hentt_tables *, const InvIO &, uint32_t, bool, hipStream_t);
struct TrCand {
  tr_fn fn;
  uint32_t ec;        // column stages (0: whole)
  const char *desc;
};

// Candidate lists per log_n (candidate 0 = default).  Defaults, from a sweep of
// whole transforms and of one to eight column stages at 1, 8 and 64 batch entries
// of 16 limbs: whole up to 2^13 (55 us against 65 with a column pass, 64
// entries); at 2^14 six column stages take 24 us against 28 whole at 8 entries
// and the same 102 us at 64; above, six to eight stages through LDS and
// one-wave blocks are 3-13% faster than five in registers (2^15: 205 against
// 217 us, 2^17 at 8 entries: 117 against 130 us).
#define W(n) {launch_whole<n>, 0, "one kernel per (batch entry, limb)"}
#define T(n, ec, e) {launch_two_pass<n, ec, e>, ec, "column stages " #ec ", block words per lane 2^" #e}
const TrCand c6[] = {W(6)}, c7[] = {W(7)}, c8[] = {W(8)}, c9[] = {W(9)}, c10[] = {W(10)}, c11[] = {W(11)},
             c12[] = {W(12)};
const TrCand c13[] = {W(13), T(13, 6, 3)};
const TrCand c14[] = {T(14, 6, 3), W(14), T(14, 2, 3)};
const TrCand c15[] = {T(15, 6, 3), T(15, 7, 3), T(15, 5, 3)};
const TrCand c16[] = {T(16, 7, 3), T(16, 8, 3), T(16, 6, 4)};
const TrCand c17[] = {T(17, 8, 3), T(17, 7, 3), T(17, 5, 3)};
#undef W
#undef T
struct TrList {
  const TrCand *c;
  uint32_t n;
};
#define L_(a) {a, (uint32_t)(sizeof(a) / sizeof(a[0]))}
const TrList k_tr[] = {L_(c6), L_(c7), L_(c8), L_(c9), L_(c10), L_(c11), L_(c12), L_(c13), L_(c14), L_(c15), L_(c16), L_(c17)};
#undef L_

}  // namespace

// ------------------------------------------------------------ tuned choices
std::atomic<uint8_t> g_choice[kTuneOps][HENTT_LOG_N_MAX + 1][kTuneClasses];

uint32_t tune_class(uint64_t units) { return units < 64 ? 0u : units < 1024 ? 1u : 2u; }

uint32_t tune_choice(int op, uint32_t log_n, uint64_t units) {
  return g_choice[op][log_n][tune_class(units)].load(std::memory_order_relaxed);
}

uint32_t transform_candidates(uint32_t log_n) { return k_tr[log_n - HENTT_LOG_N_MIN].n; }

const char *transform_describe(uint32_t log_n, uint32_t choice) { return k_tr[log_n - HENTT_LOG_N_MIN].c[choice].desc; }

uint32_t transform_cols(uint32_t log_n, uint32_t choice) { return k_tr[log_n - HENTT_LOG_N_MIN].c[choice].ec; }

static int run(const hentt_tables *t, const InvIO &io, uint32_t batch, hipStream_t st, bool inv) {
  const uint32_t ln = t->s->log_n;
  const TrList &l = k_tr[ln - HENTT_LOG_N_MIN];
  uint32_t c = tune_choice(inv ? HENTT_OP_INV : HENTT_OP_FWD, ln, (uint64_t)batch * t->limbs);
  if (c >= l.n) c = 0;
  const uint32_t piece = batch_piece(ln, t->limbs, batch);
  for (uint64_t b = 0; b < batch; b += piece)
    l.c[c].fn(t, InvIO{io.src + b * io.src_sb, io.dst + b * io.dst_sb, io.src_sb, io.dst_sb},
              (uint32_t)std::min<uint64_t>(piece, batch - b), inv, st);
  HIPCHK(hipGetLastError());
  return HENTT_OK;
}

int run_transform(const hentt_tables *t, uint64_t *x, uint32_t batch, hipStream_t st, bool inv) {
  const uint64_t sb = (uint64_t)t->limbs << t->s->log_n;
  return run(t, InvIO{x, x, sb, sb}, batch, st, inv);
}

int run_inverse_from(const hentt_tables *t, const uint64_t *src, uint64_t src_sb, uint64_t *dst, uint32_t batch,
                     hipStream_t st) {
  const uint64_t sb = (uint64_t)t->limbs << t->s->log_n;
  return run(t, InvIO{src, dst, src_sb, sb}, batch, st, true);
}

void stage_split(uint32_t log_n, uint32_t *transform_cols, uint32_t *product_cols) {
  *transform_cols = k_tr[log_n - HENTT_LOG_N_MIN].c[0].ec;
  *product_cols = product_default_cols(log_n);
}

}  // namespace hentt_rt
