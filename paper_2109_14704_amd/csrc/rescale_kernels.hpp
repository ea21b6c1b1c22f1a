// Rescale RS (section II-A): drop the last prime qL of a level with rounding,
// c' = round(c / qL) mod q_i for the remaining limbs i.  With h = (qL - 1)/2
// and r = (c_L + h) mod qL (c_L the last limb's coefficient), the RNS form is
//   c'_i = (c_i - t_i) * qL^-1 mod q_i,   t_i = (r - h) mod q_i,
// and, the transforms being linear, the same holds in the NTT domain with
// t_i replaced by NTT_i(t_i): the last limb is inverse-transformed once, and
// for every remaining limb its t_i is forward-transformed modulo q_i with the
// reduction fused into the first load (prologue) and the subtraction and
// scaling fused into the last store (epilogue).
#pragma once
#include "ntt_kernels.hpp"

namespace hentt {

struct RsLimb {   // per remaining limb i of a level
  TwM w;          // qL^-1 mod q_i
  uint64_t mu;    // floor(2^64 / q_i)
  uint64_t nh;    // q_i - (h mod q_i)
  uint64_t off;   // a multiple of q_i above any lazy forward output (rs_epilogue)
  uint64_t pad;
};

// t_i from the last limb's canonical coefficient x (mod qL): s = (x + h) mod qL,
// then s + nh subtracts h.  The forward transform takes the 60-bit word as it
// is: without corrections (34..55 bits) it adds at most 17 12q < 2^62.7, and the
// corrected form takes any word.  Moduli of 33 or fewer bits, whose final
// reduction is bounded by 2^(k + 21), reduce s first (the estimate floor(s mu /
// 2^64) is short by at most one).
__device__ __forceinline__ uint64_t rs_prologue(uint64_t x, uint64_t qL, uint64_t h, const RsLimb &r,
                                                const NttConst &n) {
  uint64_t s = csub(x + h, qL);
  if (n.k < 34) s -= mulhi64(s, r.mu) * n.q;
  return s + r.nh;
}

// (c - t) qL^-1 mod q for canonical c and a lazy forward output t: canonical.
// off - t >= 0 and c + off < 2^64: t stays below 2^60 + 2^62.7 up to 55 bits
// (off: the multiple of q just below 2^63) and below 15q above (off = 15q).
__device__ __forceinline__ uint64_t rs_epilogue(uint64_t c, uint64_t t, const RsLimb &r, const NttConst &n,
                                                uint32_t four) {
  return reduce_word(mul_tw(r.w, (c + r.off) - t, n, four), n);
}

struct RsArgs {
  const uint64_t *c;    // [batch][L + 1][N] input (NTT or coefficient domain)
  const uint64_t *tl;   // [batch][N] last limb in the coefficient domain (NTT path; or see k_rs_cols)
  uint64_t *out;        // [batch][L][N]
  const RsLimb *rs;     // [L]
  uint64_t qL, h;
  uint32_t batch, L;
};

// Unit u of a launch: output limb i of batch entry b, limb-major so that
// neighbouring workgroups share limb i's twiddles.
__device__ __forceinline__ void rs_unit(uint32_t u, uint32_t batch, uint32_t &b, uint32_t &i) {
  i = u / batch;
  b = u % batch;
}

// Whole transform per workgroup (N <= 2^13): prologue, forward rounds,
// canonical reduction, epilogue.
template <int LOGN, int E>
__global__ __launch_bounds__(1 << (LOGN - E)) void k_rs_whole(RsArgs a, const TwM *__restrict__ tw,
                                                               const NttConst *__restrict__ lc) {
  __shared__ uint64_t lds[LdsSize<LOGN>::value];
  uint32_t b, i;
  rs_unit(blockIdx.x, a.batch, b, i);
  const NttConst c = lc[i];
  const RsLimb r = a.rs[i];
  const TwM *t = tw + (size_t)i * 2 * (1u << LOGN);
  const uint32_t tid = threadIdx.x;
  using F = FwdFirst<LOGN, E>;
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    constexpr bool FIX = decltype(FX)::value;
    uint64_t v[1 << E];
    load_global<LOGN, E, F::LO, F::R>(v, a.tl + ((uint64_t)b << LOGN), RoundMap<LOGN, E, F::LO, F::R>::lane_part(tid));
  #pragma unroll
    for (int s = 0; s < (1 << E); ++s) v[s] = rs_prologue(v[s], a.qL, a.h, r, c);
    fwd_block_rounds<LOGN, E, F::LO, F::R, FIX>(v, LOGN, lds, tid, 0, t, c);
    const uint32_t four = opaque4();
    uint64_t cv[1 << E];
    load_global_m0<LOGN, E>(cv, a.c + (((uint64_t)b * (a.L + 1) + i) << LOGN), lds, tid);
  #pragma unroll
    for (int s = 0; s < (1 << E); ++s) v[s] = rs_epilogue(cv[s], v[s], r, c, four);
    store_global_m0<LOGN, E>(v, a.out + (((uint64_t)b * a.L + i) << LOGN), lds, tid);
  });
}

// Column pass (first EC forward stages) of t_i from the last limb, into out.
// Batch-entry-major order: the L units of one batch entry read the same
// last-limb columns one after another, so all but the first read hit the
// XCD's L2 (tile t of every unit lands on the same XCD when the tile count is
// a multiple of 8), with ordinary loads: streaming ones were mostly read again
// from beyond it (N = 2^16, 24 limbs, 64 polynomials: 255 us, 227 with ordinary).
// INV: the last limb comes as the inverse transform's block pass leaves it, and
// every workgroup takes its last EC stages as well (they end in the lane map the
// forward pass begins with).  That is L times the work for one launch less.
template <int LOGN, int EC, bool INV>
__global__ __launch_bounds__(cols_lanes<EC>(), EC < 8 ? 4 : 1) void k_rs_cols(RsArgs a, const TwM *__restrict__ tw,
                                                              const NttConst *__restrict__ lc) {
  __shared__ uint64_t lds[cols_lds<EC>()];
  constexpr uint32_t tiles = cols_blocks_per_unit<LOGN, EC>();
  const uint32_t u = blockIdx.x / tiles;
  const uint32_t b = u / a.L, i = u % a.L;
  const uint32_t col = (blockIdx.x % tiles) * LC<EC> + threadIdx.x % LC<EC>;
  const uint64_t *src = a.tl + ((uint64_t)b << LOGN);
  const auto ld = [&](uint32_t row) { return gload<false>(src, (row << (LOGN - EC)) + col); };
  uint64_t x[16];
  if constexpr (INV) {
    const NttConst c = lc[a.L];
    by_class(c, [&](auto FX) __attribute__((always_inline)) {
      lcol_inv<LOGN, EC, decltype(FX)::value>(x, ld, tw + ((size_t)a.L * 2 + 1) * (1u << LOGN), c, lds);
    });
    __syncthreads();  // the LDS reads before the forward pass's writes
  } else {
    const uint32_t w = lcol_w<EC>();
#pragma unroll
    for (uint32_t r = 0; r < 16; ++r) x[r] = ld((r << (EC - 4)) + w);
  }
  const NttConst c = lc[i];
  const RsLimb r = a.rs[i];
  uint64_t *dst = a.out + (((uint64_t)b * a.L + i) << LOGN);
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    uint64_t v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = rs_prologue(x[k], a.qL, a.h, r, c);
    lcol_fwd<LOGN, EC, decltype(FX)::value>(
        v, [&](uint32_t row, uint64_t y) { gstore<true>(dst, (row << (LOGN - EC)) + col, y); },
        tw + (size_t)i * 2 * (1u << LOGN), c, lds);
  });
}

// Block pass (remaining stages) in place on out, then the epilogue.
template <int LOGN, int ST, int B, int E>
__global__ __launch_bounds__(1 << (B - E)) void k_rs_blocks(RsArgs a, const TwM *__restrict__ tw,
                                                             const NttConst *__restrict__ lc) {
  __shared__ uint64_t lds[LdsSize<B>::value];
  constexpr uint32_t tiles = 1u << (LOGN - B);
  uint32_t b, i;
  rs_unit(blockIdx.x / tiles, a.batch, b, i);
  const uint32_t blockStart = (blockIdx.x % tiles) << B;
  const NttConst c = lc[i];
  const RsLimb r = a.rs[i];
  uint64_t *p = a.out + (((uint64_t)b * a.L + i) << LOGN) + blockStart;
  const uint32_t tid = threadIdx.x;
  using F = FwdFirst<ST, E>;
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    constexpr bool FIX = decltype(FX)::value;
    uint64_t v[1 << E];
    load_global<B, E, F::LO, F::R>(v, p, RoundMap<B, E, F::LO, F::R>::lane_part(tid));
    fwd_block_rounds<B, E, F::LO, F::R, FIX>(v, LOGN, lds, tid, blockStart, tw + (size_t)i * 2 * (1u << LOGN), c);
    const uint32_t four = opaque4();
    uint64_t cv[1 << E];
    load_global_m0<B, E>(cv, a.c + (((uint64_t)b * (a.L + 1) + i) << LOGN) + blockStart, lds, tid);
  #pragma unroll
    for (int s = 0; s < (1 << E); ++s) v[s] = rs_epilogue(cv[s], v[s], r, c, four);
    store_global_m0<B, E>(v, p, lds, tid);
  });
}

// Coefficient-domain rescale: element-wise, tiles of 2048 words.
__global__ __launch_bounds__(256) void k_rs_coeff(RsArgs a, const NttConst *__restrict__ lc, uint32_t log_n,
                                                  uint32_t tiles) {
  uint32_t b, i;
  rs_unit(blockIdx.x / tiles, a.batch, b, i);
  const uint32_t n = 1u << log_n, base = (blockIdx.x % tiles) * 2048u;
  const NttConst c = lc[i];
  const RsLimb r = a.rs[i];
  const uint64_t *ci = a.c + (((uint64_t)b * (a.L + 1) + i) << log_n);
  const uint64_t *cl = a.c + (((uint64_t)b * (a.L + 1) + a.L) << log_n);
  uint64_t *o = a.out + (((uint64_t)b * a.L + i) << log_n);
  const uint32_t four = opaque4();
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const uint32_t k = base + threadIdx.x + 256u * s;
    if (k < n) o[k] = rs_epilogue(ci[k], est3(rs_prologue(cl[k], a.qL, a.h, r, c), c), r, c, four);
  }
}

}  // namespace hentt
