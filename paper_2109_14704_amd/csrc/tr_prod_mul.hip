// Compiled instances of the dyadic product and the fused negacyclic polymul at
// every N (candidate 0 is the default and serves every domain combination),
// and the common entry of both product kinds.
#include <algorithm>

#include "prod_launch.hpp"

namespace hentt_rt {
namespace {
#define D(n, pec, e) {launch_prod_cfg<n, PROD_MUL, pec, e, true>, pec, "column stages " #pec ", block words per lane 2^" #e}
#define C(n, pec, e) {launch_prod_cfg<n, PROD_MUL, pec, e, false>, pec, "column stages " #pec ", block words per lane 2^" #e}
const ProdCand m6[] = {D(6, 0, 2)}, m7[] = {D(7, 0, 2)}, m8[] = {D(8, 0, 2)}, m9[] = {D(9, 0, 2)},
               m10[] = {D(10, 0, 2)}, m11[] = {D(11, 0, 3)}, m12[] = {D(12, 0, 3)};
const ProdCand m13[] = {D(13, 6, 3), C(13, 0, 3)};
const ProdCand m14[] = {D(14, 6, 3), C(14, 7, 2)};
const ProdCand m15[] = {D(15, 6, 3), C(15, 7, 3)};
const ProdCand m16[] = {D(16, 7, 3), C(16, 8, 3)};
const ProdCand m17[] = {D(17, 8, 3), C(17, 7, 3)};
#undef D
#undef C
const ProdList k_mul[] = {HENTT_PROD_LIST(m6),  HENTT_PROD_LIST(m7),  HENTT_PROD_LIST(m8),  HENTT_PROD_LIST(m9),
                          HENTT_PROD_LIST(m10), HENTT_PROD_LIST(m11), HENTT_PROD_LIST(m12), HENTT_PROD_LIST(m13),
                          HENTT_PROD_LIST(m14), HENTT_PROD_LIST(m15), HENTT_PROD_LIST(m16), HENTT_PROD_LIST(m17)};
}  // namespace

const ProdCand *prod_candidates(int mode, uint32_t log_n, uint32_t *count) {
  if (mode == PROD_TENSOR) return tensor_candidates(log_n, count);
  const ProdList &l = k_mul[log_n - HENTT_LOG_N_MIN];
  *count = l.n;
  return l.c;
}

uint32_t product_default_cols(uint32_t log_n) { return k_mul[log_n - HENTT_LOG_N_MIN].c[0].pec; }

const ProdCand &prod_select(int mode, uint32_t log_n, uint64_t units, bool fused) {
  uint32_t n = 0;
  const ProdCand *c = prod_candidates(mode, log_n, &n);
  // the NTT-domain forms run the default instance
  uint32_t i = fused ? tune_choice(mode == PROD_MUL ? HENTT_OP_POLYMUL : HENTT_OP_TENSOR, log_n, units) : 0;
  if (i == 0 && mode == PROD_TENSOR && log_n == 9 && tensor9_one_wave(units)) i = 1;
  return c[i < n ? i : 0];
}

// The instance that needs no workspace, for the fused product of the sizes that
// have one beside a two-pass default (2^13), else null.
static const ProdCand *whole_instance(int mode, uint32_t log_n) {
  uint32_t n = 0;
  const ProdCand *c = prod_candidates(mode, log_n, &n);
  for (uint32_t i = 0; i < n; ++i)
    if (c[i].pec == 0) return c + i;
  return nullptr;
}

// Whether the fused product at 2^13 runs whole where no instance was chosen.  A whole
// one fills a CU, so calls take 32 us (38 with 60-bit moduli) per generation of as
// many units as the chip has CUs; the two-pass default takes time in proportion, 0.13
// us a unit.  Measured on 256 CUs, two-pass and whole, 55 bits (60 bits): 128 units 26.2
// and 26.5 (29.5, 32.0), 256 45.4 and 32.1 (50.4, 38.6), 264 49.7 and 55.4 (56.5, 67.2),
// 512 78 and 65 (88, 76), 640 87 and 82 (96, 98), 704 97 and 83 (106, 99), 1120 138 and 134
// (152, 161), 4096 464 and 423 (518, 511): whole where the last generation is full or
// more than half full.
static bool whole_fits(uint64_t units, uint32_t cus) {
  const uint64_t last = units % cus;
  return last == 0 || 2 * last > cus;
}

int run_prod(const hentt_tables *t, int mode, const ProdArgs &pa, uint32_t batch, bool in_coeff, bool out_coeff,
             hipStream_t st) {
  const uint32_t ln = t->s->log_n;
  const int nin = mode == PROD_MUL ? 2 : 4;
  const uint64_t NL = (uint64_t)t->limbs << ln, units = (uint64_t)batch * t->limbs;
  const ProdCand *c = &prod_select(mode, ln, units, in_coeff && out_coeff);
  const ProdCand *whole = in_coeff && out_coeff && c->pec > 0 ? whole_instance(mode, ln) : nullptr;
  if (whole && whole_fits(units, t->s->cus)) c = whole;
  const uint32_t piece = batch_piece(ln, t->limbs, batch);
  void *ws = nullptr;
  if (in_coeff && c->pec > 0) {
    // Where a whole instance exists, the workspace only makes the call faster: it is
    // not allocated into a capture (which an allocation would end), and done without
    // when it cannot be had.
    int rc = pool_get((size_t)nin * piece * NL * 8ull, st, &ws, !whole || !capturing(st));
    if (rc == HENTT_ENOMEM && whole) c = whole;
    else if (rc) return rc;
  }
  for (uint64_t b = 0; b < batch; b += piece) {
    ProdArgs pb = pa;
    for (int p = 0; p < nin; ++p) pb.in[p] += b * pa.in_sb;
    for (int o = 0; o < (mode == PROD_MUL ? 1 : 3); ++o) pb.out[o] += b * pa.out_sb;
    c->fn(t, pb, (uint32_t)std::min<uint64_t>(piece, batch - b), in_coeff, out_coeff, (uint64_t *)ws, st);
  }
  hipError_t e = hipGetLastError();
  if (ws) pool_put(ws);
  if (e != hipSuccess) return hip_fail(e);
  return HENTT_OK;
}

}  // namespace hentt_rt
