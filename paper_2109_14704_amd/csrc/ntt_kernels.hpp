// Staged negacyclic NTT kernels for gfx950 (CDNA4), section III-B of the paper
// re-planned for a 64-wide wavefront, a 160 KB LDS and 512 VGPRs per lane.
//
// Data: x[poly][N] uint64, poly = batch * limbs + limb (limb fastest among
// polynomials, coefficient fastest overall).  Twiddles per limb: forward table
// psi^brv(k) and inverse table psi^-brv(k), k < N, each a 16-byte TwM word
// (modarith.hpp).
//
// A transform is a sequence of "rounds".  A round applies R consecutive
// butterfly stages to groups of 2^R elements held in one lane's registers;
// the butterfly pairs of those stages differ in the index bits
// [LO, LO + R).  Rounds exchange data through LDS (inside a workgroup) or
// through HBM (between the column pass and the block pass of large N), as in
// the staged global -> local -> register design of section III-B, with the
// radix-2^R register blocking of its high-radix subsection.
#pragma once
#include <type_traits>

#include "modarith.hpp"
#include "schedule.hpp"

namespace hentt {

// LDS padding: one spare element after every 16.  Made for rounds of 16 words per
// lane, whose strided accesses it puts on distinct banks; with 8 and 4 words some
// still meet (SQ_LDS_BANK_CONFLICT of SQ_LDS_IDX_ACTIVE: the tensor's block kernel
// at 2^16 48.8 M of 132 M cycles, the polymul's at 2^15 27.3 M of 75.5 M, the
// persistent batch 9% forward and 22% inverse).  Column passes through LDS have a
// layout of their own and no conflicts.
__device__ __forceinline__ constexpr uint32_t lds_pad(uint32_t i) { return i + (i >> 4); }
template <int B> struct LdsSize { static constexpr int value = (1 << B) + (1 << B) / 16; };

// Which block index bits a lane owns in a round over bits [LO, LO+R) of a
// block of 2^B elements, with 2^E elements per lane (E >= R), 2^(B-E) lanes.
// Lane bits fill the lowest free positions (coalescing), the remaining
// E - R "group" bits the rest.
template <int B, int E, int LO, int R>
struct RoundMap {
  static_assert(E >= R && LO + R <= B && E <= B, "bad round");
  static constexpr int TB = B - E;
  static constexpr bool LANE_LOW = (TB <= LO);  // all lane bits below LO: twiddles uniform per block
  __device__ static __forceinline__ uint32_t lane_part(uint32_t tid) {
    if constexpr (LANE_LOW) return tid;
    else return (tid & ((1u << LO) - 1)) | ((tid >> LO) << (LO + R));
  }
  static constexpr uint32_t g_part(int g) {
    uint32_t r = 0;
    int bit = 0;
    if constexpr (LANE_LOW) {
      for (int pos = TB; pos < LO; ++pos, ++bit) if ((g >> bit) & 1) r |= 1u << pos;
      for (int pos = LO + R; pos < B; ++pos, ++bit) if ((g >> bit) & 1) r |= 1u << pos;
    } else {
      for (int pos = TB + R; pos < B; ++pos, ++bit) if ((g >> bit) & 1) r |= 1u << pos;
    }
    return r;
  }
  static constexpr uint32_t slot_part(int s) { return g_part(s >> R) | (uint32_t)((s & ((1 << R) - 1)) << LO); }
};

// Twiddle tables are never written while a kernel runs, so they are read
// through the constant address space: a wave-uniform index becomes a scalar
// load even when the table pointer was itself read from memory.
__device__ __forceinline__ TwM ld_tw(const TwM* t, uint32_t i) {
  const __attribute__((address_space(4))) uint64_t* p = (const __attribute__((address_space(4))) uint64_t*)(t + i);
  const uint64_t a = p[0], b = p[1];
  return TwM{lo32(a), hi32(a), lo32(b), hi32(b)};
}

// Returns p unchanged but hides that from the optimiser (adds an opaque,
// wave-uniform zero), so loads through it are not merged with earlier ones.
template <typename T> __device__ __forceinline__ const T *opaque(const T *p) {
  uint32_t z = 0;
  asm volatile("" : "+s"(z));
  return p + z;
}

// Limb constants through the constant address space as well: with a
// wave-uniform pointer (also one read from memory) they become scalar loads
// into SGPRs instead of 24 VGPRs of per-lane copies.
__device__ __forceinline__ NttConst ld_nc(const NttConst *p) {
  const __attribute__((address_space(4))) uint64_t *w = (const __attribute__((address_space(4))) uint64_t *)p;
  NttConst c;
  c.q = w[0];
  c.nq = w[1];
  c.mu = w[2];
  c.off = w[3];
  c.qlo = lo32(w[4]);
  c.qhi = hi32(w[4]);
  c.qi = lo32(w[5]);
  c.k = hi32(w[5]);
  c.c64 = lo32(w[6]);
  c.ce = hi32(w[6]);
  c.s0 = lo32(w[7]);
  c.s1 = hi32(w[7]);
  c.ninv = TwM{lo32(w[8]), hi32(w[8]), lo32(w[9]), hi32(w[9])};
  c.ninvw = TwM{lo32(w[10]), hi32(w[10]), lo32(w[11]), hi32(w[11])};
  return c;
}

// Compile-time loop: f(std::integral_constant<int, I>) for I in [I0, I1), so
// that array indices stay constants (no stack arrays) even for loop bodies too
// large for the unroller.
template <int I0, int I1, typename F> __device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I0 < I1) {
    f(std::integral_constant<int, I0>{});
    static_for<I0 + 1, I1>(f);
  }
}

// Moduli of 34 to 55 bits run without corrections inside the rounds (schedule.hpp);
// the others (FIX) take theirs unconditionally.  A kernel holds both forms of its
// body and branches once, on its workgroup's limb.  Tests at every stage
// instead cut the body into blocks that the scheduler could not overlap and
// roughly doubled its registers (k_cols of five stages 260 VGPRs against 103);
// the markers keep the compiler from merging the two forms' heads and tails,
// which did the same.
template <typename F> __device__ __forceinline__ void by_class(const NttConst &c, F &&f) {
  if (uncorrected(c.k)) {
    asm volatile("; class 0");
    f(std::false_type{});
    asm volatile("; end 0");
  } else {
    asm volatile("; class 1");
    f(std::true_type{});
    asm volatile("; end 1");
  }
}

// ---------------------------------------------------------------- rounds --
// Forward stages with global index s = LOGN - LO - R + u, u < R.  Stage s
// pairs j with j + N/2^(s+1) and uses psi_rev[2^s + (j >> (LOGN - s))].
// Bounds and corrections: schedule.hpp.
template <int B, int E, int LO, int R, bool FIX, bool PRE = false>
__device__ __forceinline__ void fwd_round(uint64_t (&x)[1 << E], uint32_t logn, uint32_t blockStart,
                                          uint32_t lanePart, const TwM* __restrict__ tw, const NttConst &c,
                                          const TwM *pf = nullptr) {
  using M = RoundMap<B, E, LO, R>;
  const uint32_t four = opaque4();
  static_for<0, R>([&](auto U) __attribute__((always_inline)) {
    constexpr int u = decltype(U)::value, h = 1 << (R - 1 - u);
    if constexpr (FIX) {
#pragma unroll
      for (int i = 0; i < (1 << E); ++i)
        if (!(i & h)) x[i] = est3(x[i], c);
    }
#pragma unroll
    for (int g = 0; g < (1 << (E - R)); ++g) {
      const uint32_t J0 = M::LANE_LOW ? (blockStart | M::g_part(g)) : (blockStart | lanePart | M::g_part(g));
      // stage s = logn - LO - R + u: 2^s = 2^(logn - B) * 2^(B - LO - R + u)
      const uint32_t base = ((1u << (logn - B)) << (B - LO - R + u)) + (J0 >> (LO + R - u));
#pragma unroll
      for (int k = 0; k < (1 << R); ++k) {
        if (k & h) continue;
        const TwM w = PRE ? pf[(1 << u) - 1 + (k >> (R - u))] : ld_tw(tw, base + (k >> (R - u)));
        ct_bfly_m(x[(g << R) + k], x[(g << R) + k + h], w, c, four);
      }
    }
  });
}
// Inverse stages v = LO + u.  Stage v pairs j with j + 2^v and uses
// psi_rev^-1[N/2^(v+1) + (j >> (v+1))].  The last stage (v = LOGN-1) also
// multiplies both outputs by N^-1.  Bounds and corrections: schedule.hpp.
template <int B, int E, int LO, int R, int LBIN, int LBOUT, bool FIX, bool PRE = false>
__device__ __forceinline__ void inv_round(uint64_t (&x)[1 << E], uint32_t logn, uint32_t blockStart,
                                           uint32_t lanePart, const TwM* __restrict__ itw, const NttConst& c,
                                           const TwM* pf = nullptr) {
  using M = RoundMap<B, E, LO, R>;
  static_assert(LBIN + R <= 9, "words stay below 512q inside a round");
  const uint32_t four = opaque4();
  static_for<0, R>([&](auto U) __attribute__((always_inline)) {
    constexpr int u = decltype(U)::value, v = LO + u, d = 1 << u;
    const uint64_t off = c.q << inv_off_log(c.k, FIX, LBIN, u, v);
    // only the block's top stage can be the transform's last one
    if (LO + u == B - 1 && (uint32_t)v == logn - 1) {
      // last stage: one group, twiddle psi^-brv(1) folded with N^-1
#pragma unroll
      for (int i = 0; i < (1 << E); ++i) {
        if (i & d) continue;
        const uint64_t s = x[i] + x[i + d], df = (x[i] + off) - x[i + d];
        x[i] = mul_tw(c.ninv, s, c, four);
        x[i + d] = mul_tw(c.ninvw, df, c, four);
      }
    } else {
#pragma unroll
      for (int g = 0; g < (1 << (E - R)); ++g) {
        const uint32_t J0 = M::LANE_LOW ? (blockStart | M::g_part(g)) : (blockStart | lanePart | M::g_part(g));
        const uint32_t base = ((1u << logn) >> (v + 1)) + (J0 >> (v + 1));
#pragma unroll
        for (int k = 0; k < (1 << R); ++k) {
          if (k & d) continue;
          const TwM w = PRE ? pf[(1 << (R - 1 - u)) - 1 + (k >> (u + 1))] : ld_tw(itw, base + (k >> (u + 1)));
          gs_bfly_m(x[(g << R) + k], x[(g << R) + k + d], w, off, c, four);
        }
      }
      if constexpr (FIX) {
#pragma unroll
        for (int i = 0; i < (1 << E); ++i)
          if (inv_fix(R, u, i & d)) x[i] = est3(x[i], c);
      } else if (u == R - 1) {
#pragma unroll
        for (int i = 0; i < (1 << E); ++i)
          if (inv_over<R, LBIN, LBOUT>(i & ((1 << R) - 1))) x[i] = est3(x[i], c);
      }
    }
  });
}
// ------------------------------------------------------------ data moves --
// Polynomial words are addressed as a base pointer plus a 32-bit byte offset
// (every index below lies inside one polynomial or block, < 2^17 words), in
// the global address space.  The compiler then issues global loads with one
// base for the wave and one 32-bit offset per lane, instead of a flat load
// with a 64-bit address per element, which matters where the base pointer
// was itself read from memory (the persistent batch kernel).
//
// NT: non-temporal (streaming) accesses, chosen per kernel by measurement:
// the column passes stream both ways (each word is read and written once, and
// the next pass over it comes after the whole batch has gone through the
// caches: 10-18% faster), the fused product kernels stream their loads (2-4%
// faster).  The block and whole-transform kernels, and the persistent batch
// kernel (which reads pass-1 results back from L2), were slower with
// streaming accesses (the forward block pass at N = 2^15 took twice as long)
// and use ordinary ones.
#define HENTT_GLOBAL __attribute__((address_space(1)))
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
template <bool NT> __device__ __forceinline__ uint64_t gload(const uint64_t* base, uint32_t i) {
  const HENTT_GLOBAL uint64_t* p = (const HENTT_GLOBAL uint64_t*)((const HENTT_GLOBAL char*)base + (i << 3));
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT> __device__ __forceinline__ void gstore(uint64_t* base, uint32_t i, uint64_t v) {
  HENTT_GLOBAL uint64_t* p = (HENTT_GLOBAL uint64_t*)((HENTT_GLOBAL char*)base + (i << 3));
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

template <int B, int E, int LO, int R, bool NT = false>
__device__ __forceinline__ void load_global(uint64_t (&x)[1 << E], const uint64_t* __restrict__ src, uint32_t lp) {
  using M = RoundMap<B, E, LO, R>;
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) x[s] = gload<NT>(src, lp + M::slot_part(s));
}
template <int B, int E, int LO, int R, bool NT = false>
__device__ __forceinline__ void store_global(const uint64_t (&x)[1 << E], uint64_t* __restrict__ dst, uint32_t lp) {
  using M = RoundMap<B, E, LO, R>;
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) gstore<NT>(dst, lp + M::slot_part(s), x[s]);
}
template <int B, int E, int LO, int R>
__device__ __forceinline__ void load_lds(uint64_t (&x)[1 << E], const uint64_t* lds, uint32_t lp) {
  using M = RoundMap<B, E, LO, R>;
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) x[s] = lds[lds_pad(lp + M::slot_part(s))];
}
template <int B, int E, int LO, int R>
__device__ __forceinline__ void store_lds(const uint64_t (&x)[1 << E], uint64_t* lds, uint32_t lp) {
  using M = RoundMap<B, E, LO, R>;
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) lds[lds_pad(lp + M::slot_part(s))] = x[s];
}

// Global stores and loads of the (0, E) map, in which every lane holds 2^E
// consecutive words, routed through LDS: the global side uses the map whose
// lanes own the lowest block bits, so that each memory instruction covers
// consecutive words across the lanes instead of one word every 2^E.  Both
// begin with a barrier (the workgroup's earlier LDS reads are done); the load
// also ends with one, so that the caller may write LDS next.
#ifndef HENTT_TS
#define HENTT_TS 1
#endif
#ifndef HENTT_TL
#define HENTT_TL 1
#endif
template <int B, int E, bool NT = false>
__device__ __forceinline__ void store_global_m0(uint64_t (&x)[1 << E], uint64_t* __restrict__ dst, uint64_t* lds,
                                                uint32_t tid) {
#if HENTT_TS
  using MT = RoundMap<B, E, B - E, E>;
  __syncthreads();
  store_lds<B, E, 0, E>(x, lds, RoundMap<B, E, 0, E>::lane_part(tid));
  __syncthreads();
  load_lds<B, E, B - E, E>(x, lds, MT::lane_part(tid));
  store_global<B, E, B - E, E, NT>(x, dst, MT::lane_part(tid));
#else
  store_global<B, E, 0, E, NT>(x, dst, RoundMap<B, E, 0, E>::lane_part(tid));
#endif
}
template <int B, int E, bool NT = false>
__device__ __forceinline__ void load_global_m0(uint64_t (&x)[1 << E], const uint64_t* __restrict__ src, uint64_t* lds,
                                               uint32_t tid) {
#if HENTT_TL
  using MT = RoundMap<B, E, B - E, E>;
  load_global<B, E, B - E, E, NT>(x, src, MT::lane_part(tid));
  __syncthreads();
  store_lds<B, E, B - E, E>(x, lds, MT::lane_part(tid));
  __syncthreads();
  load_lds<B, E, 0, E>(x, lds, RoundMap<B, E, 0, E>::lane_part(tid));
  __syncthreads();
#else
  load_global<B, E, 0, E, NT>(x, src, RoundMap<B, E, 0, E>::lane_part(tid));
#endif
}

// The same load for a workgroup whose LDS holds nothing yet (the first
// access of a kernel or of a persistent tile): direct global-to-LDS loads
// (global_load_lds_dwordx4), which move each lane's 16 bytes into the wave's
// 1 KB LDS window without passing through registers, then one 16-byte LDS
// read per word pair.  One instruction fills a contiguous window, so the LDS
// layout is set by which global pair each lane fetches: pair P = 8t + k of
// the block sits at LDS pair 8t + (k ^ (t mod 8)) (the map is its own
// inverse), which puts the eight pairs one 8-lane group reads in eight
// different 16-byte bank groups.  Ends with a barrier, like load_global_m0.
//
// Data need only be 8-byte aligned.  The 16-byte form moves 16-byte units, so
// where src is not one (uniform per workgroup) four 4-byte loads (at four
// times the instructions) fill the same layout dword by dword.  Taking
// load_global_m0 there instead cost registers on the aligned path: 69 for 56
// in the whole 2^11 and 2^12 inverse, 24 spilled in the persistent batch's.
#ifndef HENTT_DMA_LOAD
#define HENTT_DMA_LOAD 1
#endif
__device__ __forceinline__ uint32_t dma_swz(uint32_t pair) { return pair ^ ((pair >> 3) & 7u); }
template <int B, int E>
__device__ __forceinline__ void load_global_m0_fresh(uint64_t (&x)[1 << E], const uint64_t* __restrict__ src,
                                                     uint64_t* lds, uint32_t tid) {
  constexpr uint32_t LANES = 1u << (B - E);
  if constexpr (HENTT_DMA_LOAD && LANES % 64 == 0 && E >= 1) {
    constexpr uint32_t WAVE_WORDS = 64u << E;   // the words one wave moves
    const uint32_t wave = tid >> 6, lane = tid & 63;
    typedef __attribute__((address_space(3))) void lds_void;
    if ((__builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)src) & 15) == 0) {
#pragma unroll
      for (uint32_t i = 0; i < WAVE_WORDS / 128; ++i) {
        const uint32_t win = wave * WAVE_WORDS + 128 * i;   // first word of this instruction's window
        const uint32_t pair = win / 2 + lane;                  // LDS pair this lane fills
        __builtin_amdgcn_global_load_lds(src + 2 * dma_swz(pair), (lds_void*)(lds + win), 16, 0, 0);
      }
    } else {
#pragma unroll 1
      for (uint32_t i = 0; i < WAVE_WORDS / 32; ++i) {
        const uint32_t win = wave * WAVE_WORDS + 32 * i;    // 64 dwords: 16 pairs
        const uint32_t pair = win / 2 + (lane >> 2);           // LDS pair this lane fills a quarter of
        __builtin_amdgcn_global_load_lds((const uint32_t*)src + 4 * dma_swz(pair) + (lane & 3), (lds_void*)(lds + win), 4,
                                         0, 0);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < (1u << (E - 1)); ++j) {
      const u64x2 w = *(const u64x2*)(lds + 2 * dma_swz((tid << (E - 1)) + j));
      x[2 * j] = w.x;
      x[2 * j + 1] = w.y;
    }
    __syncthreads();
  } else {
    load_global_m0<B, E>(x, src, lds, tid);
  }
}

// Canonical reduction of a transform's outputs.
template <int E, bool FIX> __device__ __forceinline__ void reduce_out(uint64_t (&x)[1 << E], const NttConst &c) {
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) {
    if constexpr (FIX) x[s] = reduce_word(x[s], c);
    else x[s] = csubn(reduce_est(x[s], c.nq, c.ce, c.k - 33), c.nq);
  }
}

// --------------------------------------------------- block transforms ----
// Forward rounds over the block bits [0, LO+R) (the first round covers
// [LO, LO+R)), starting from registers already loaded with the first round's
// map.  Ends with the lane holding the last round (LO = 0) map in registers,
// i.e. 2^E consecutive elements, lazy values (see fwd_round).
//
// PRE: a round's twiddles (2^R - 1 root powers per lane) are loaded ahead of the
// LDS exchange in front of it, so that their latency runs beside the barrier and
// not after it, and once per round instead of in two groups as registers allow.
// HAVE: this round's are in pf.  Used where the registers it takes (84 -> 112 for
// the whole 2^12, 95 for blocks) cost no occupancy that counts, the polymul of 2^10
// and more: 2^12, one product, 12.7 -> 12.2 us; 512 x 8 limbs 196 -> 192; 2^10, 2048
// x 8 limbs 171 -> 161; the blocks of 128 x 16 limbs at 2^15 3% less.  The tensor's
// and the key switch's blocks stand at 128 registers without it.
template <int B, int E, int LO, int R, bool FIX, bool PRE = false, bool HAVE = false>
__device__ __forceinline__ void fwd_block_rounds(uint64_t (&x)[1 << E], uint32_t logn, uint64_t* lds, uint32_t tid,
                                                 uint32_t blockStart, const TwM* __restrict__ tw, const NttConst &c,
                                                 const TwM *pf = nullptr) {
  using M = RoundMap<B, E, LO, R>;
  const uint32_t lp = M::lane_part(tid);
  fwd_round<B, E, LO, R, FIX, HAVE>(x, logn, blockStart, lp, tw, c, pf);
  if constexpr (LO > 0) {
    constexpr int R2 = E;
    constexpr int LO2 = LO - R2;
    static_assert(LO2 >= 0, "rounds must tile the block");
    using M2 = RoundMap<B, E, LO2, R2>;
    TwM w[PRE ? (1 << R2) - 1 : 1];
    if constexpr (PRE) {
#pragma unroll
      for (int u = 0; u < R2; ++u) {
        const uint32_t base = ((1u << (logn - B)) << (B - LO2 - R2 + u)) + ((blockStart | M2::lane_part(tid)) >> (LO2 + R2 - u));
#pragma unroll
        for (int i = 0; i < (1 << u); ++i) w[(1 << u) - 1 + i] = ld_tw(tw, base + i);
      }
    }
    store_lds<B, E, LO, R>(x, lds, lp);
    __syncthreads();
    load_lds<B, E, LO2, R2>(x, lds, M2::lane_part(tid));
    fwd_block_rounds<B, E, LO2, R2, FIX, PRE, PRE>(x, logn, lds, tid, blockStart, tw, c, w);
  }
}

// Inverse rounds over block bits [LO, ST), starting from registers loaded with
// the (LO, R) map; ST < B when the lanes of a workgroup hold several blocks of
// 2^ST words side by side.  Ends with the lane holding the last round's map
// (covering [ST - Rlast, ST)); words enter below 16q and leave below 16q, or
// are the transform's lazy outputs.
template <int B, int ST, int E, int LO, int R, bool FIX, bool PRE = false, bool HAVE = false>
__device__ __forceinline__ void inv_block_rounds(uint64_t (&x)[1 << E], uint32_t logn, uint64_t* lds, uint32_t tid,
                                                 uint32_t blockStart, const TwM* __restrict__ itw,
                                                 const NttConst& c, const TwM* pf = nullptr) {
  using M = RoundMap<B, E, LO, R>;
  const uint32_t lp = M::lane_part(tid);
  inv_round<B, E, LO, R, LB_ROUND, (LO + R < ST ? LB_ROUND : LB_PASS), FIX, HAVE>(x, logn, blockStart, lp, itw, c, pf);
  if constexpr (LO + R < ST) {
    constexpr int LO2 = LO + R;
    constexpr int R2 = (ST - LO2) < E ? (ST - LO2) : E;
    using M2 = RoundMap<B, E, LO2, R2>;
    constexpr bool AHEAD = PRE && R2 == E && !M2::LANE_LOW;
    TwM w[AHEAD ? (1 << R2) - 1 : 1];
    if constexpr (AHEAD) {
#pragma unroll
      for (int u = 0; u < R2; ++u) {
        const uint32_t base = ((1u << logn) >> (LO2 + u + 1)) + ((blockStart | M2::lane_part(tid)) >> (LO2 + u + 1));
#pragma unroll
        for (int i = 0; i < (1 << (R2 - 1 - u)); ++i) w[(1 << (R2 - 1 - u)) - 1 + i] = ld_tw(itw, base + i);
      }
    }
    store_lds<B, E, LO, R>(x, lds, lp);
    __syncthreads();
    load_lds<B, E, LO2, R2>(x, lds, M2::lane_part(tid));
    inv_block_rounds<B, ST, E, LO2, R2, FIX, PRE, AHEAD>(x, logn, lds, tid, blockStart, itw, c, w);
  }
}

// Map blockIdx -> (polynomial, tile): limb-major, batch next, tile fastest, so
// that concurrently running workgroups share one limb's twiddle table in L2.
struct Unit {
  uint32_t poly, b, limb, tile;
};
__device__ __forceinline__ Unit unit_of(uint32_t bid, uint32_t tiles, uint32_t batch, uint32_t limbs) {
  Unit u;
  u.tile = bid % tiles;
  uint32_t r = bid / tiles;
  u.limb = r / batch;
  u.b = r % batch;
  u.poly = u.b * limbs + u.limb;
  return u;
}

// ------------------------------------------------------------- kernels ----
// Whole transform of one polynomial per workgroup (N = 2^LOGN fits in LDS).
template <int LOGN, int E>
__global__ __launch_bounds__(1 << (LOGN - E), LOGN == 13 && E == 4 ? 4 : 1) void k_fwd_whole(uint64_t* __restrict__ x, const TwM* __restrict__ tw,
                                                                const NttConst* __restrict__ lc, uint32_t batch,
                                                                uint32_t limbs) {
  __shared__ __attribute__((aligned(16))) uint64_t lds[LdsSize<LOGN>::value];
  const Unit un = unit_of(blockIdx.x, 1, batch, limbs);
  const NttConst c = lc[un.limb];
  const TwM* t = tw + (size_t)un.limb * 2 * (1u << LOGN);
  uint64_t* p = x + (size_t)un.poly * (1u << LOGN);
  const uint32_t tid = threadIdx.x;
  using F = FwdFirst<LOGN, E>;
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    constexpr bool FIX = decltype(FX)::value;
    uint64_t v[1 << E];
    load_global<LOGN, E, F::LO, F::R>(v, p, RoundMap<LOGN, E, F::LO, F::R>::lane_part(tid));
    fwd_block_rounds<LOGN, E, F::LO, F::R, FIX>(v, LOGN, lds, tid, 0, t, c);
    reduce_out<E, FIX>(v, c);
    store_global_m0<LOGN, E>(v, p, lds, tid);
  });
}

// Batch of an inverse transform: limb l of entry b is read at src + b src_sb +
// l N and its first pass written to dst + b dst_sb + l N (equal for in place).
struct InvIO {
  const uint64_t* src;
  uint64_t* dst;
  uint64_t src_sb, dst_sb;  // words between consecutive batch entries
};

template <int LOGN, int E>
__global__ __launch_bounds__(1 << (LOGN - E)) void k_inv_whole(InvIO io, const TwM* __restrict__ tw,
                                                                const NttConst* __restrict__ lc, uint32_t batch,
                                                                uint32_t limbs) {
  __shared__ __attribute__((aligned(16))) uint64_t lds[LdsSize<LOGN>::value];
  const Unit un = unit_of(blockIdx.x, 1, batch, limbs);
  const NttConst c = lc[un.limb];
  const TwM* it = tw + ((size_t)un.limb * 2 + 1) * (1u << LOGN);
  const uint64_t* src = io.src + un.b * io.src_sb + ((uint64_t)un.limb << LOGN);
  uint64_t* dst = io.dst + un.b * io.dst_sb + ((uint64_t)un.limb << LOGN);
  const uint32_t tid = threadIdx.x;
  using L = InvLast<LOGN, E>;
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    constexpr bool FIX = decltype(FX)::value;
    uint64_t v[1 << E];
    load_global_m0_fresh<LOGN, E>(v, src, lds, tid);
    inv_block_rounds<LOGN, LOGN, E, 0, (LOGN < E ? LOGN : E), FIX>(v, LOGN, lds, tid, 0, it, c);
    reduce_out<E, FIX>(v, c);
    store_global<LOGN, E, L::LO, L::R>(v, dst, RoundMap<LOGN, E, L::LO, L::R>::lane_part(tid));
  });
}

// Column pass: the first E forward stages (or the last E inverse stages) on
// 2^E elements at stride N / 2^E; workgroup of 256 lanes = 256 columns.
// Twiddles are the same for every lane (scalar loads).  Up to four
// polynomial sets ("components") per launch, each read from src[c] and
// written to dst[c] (equal for in place).
struct ColArgs {
  const uint64_t *src[4];
  uint64_t *dst[4];
  uint64_t src_sb, dst_sb;  // words between consecutive batch entries
};

// One column of the column pass: 2^E elements at stride N / 2^E starting at
// word `col`, read from src and written to dst (equal for in place).  `t` is
// the limb's forward table, or its inverse table when INV.
template <int LOGN, int E, bool INV, bool FIX>
__device__ __forceinline__ void col_pass(const uint64_t *src, uint64_t *dst, uint32_t col, const TwM *t,
                                         const NttConst &c) {
  constexpr int LO = LOGN - E;
  uint64_t v[1 << E];
  load_global<LOGN, E, LO, E, true>(v, src, col);
  if constexpr (!INV) {
    fwd_round<LOGN, E, LO, E, FIX>(v, LOGN, 0, col, t, c);
  } else {
    inv_round<LOGN, E, LO, E, LB_PASS, LB_PASS, FIX>(v, LOGN, 0, col, t, c);
    reduce_out<E, FIX>(v, c);
  }
  store_global<LOGN, E, LO, E, true>(v, dst, col);
}

// Columns per lane: two neighbouring columns (16-byte accesses) for passes of
// up to 16 words per lane; at 32 words per lane the doubled registers cost
// more than the wider accesses gain (measured: column passes of 2^17
// transforms 12% faster, of the 2^15 and 2^16 products 6-10% slower).
template <int E> struct ColCpl { static constexpr int value = E <= 4 ? 2 : 1; };
// Two neighbouring columns per lane: 16-byte accesses.
template <int LOGN, int E, bool INV, bool FIX>
__device__ __forceinline__ void col_pass2(const uint64_t *src, uint64_t *dst, uint32_t col, const TwM *t,
                                          const NttConst &c) {
  constexpr int LO = LOGN - E;
  uint64_t v0[1 << E], v1[1 << E];
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) {
    const HENTT_GLOBAL u64x2 *p = (const HENTT_GLOBAL u64x2 *)((const HENTT_GLOBAL char *)src + ((col + (s << LO)) << 3));
    const u64x2 w = __builtin_nontemporal_load(p);
    v0[s] = w.x;
    v1[s] = w.y;
  }
  if constexpr (!INV) {
    fwd_round<LOGN, E, LO, E, FIX>(v0, LOGN, 0, col, t, c);
    fwd_round<LOGN, E, LO, E, FIX>(v1, LOGN, 0, col, t, c);
  } else {
    inv_round<LOGN, E, LO, E, LB_PASS, LB_PASS, FIX>(v0, LOGN, 0, col, t, c);
    inv_round<LOGN, E, LO, E, LB_PASS, LB_PASS, FIX>(v1, LOGN, 0, col, t, c);
    reduce_out<E, FIX>(v0, c);
    reduce_out<E, FIX>(v1, c);
  }
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) {
    HENTT_GLOBAL u64x2 *p = (HENTT_GLOBAL u64x2 *)((HENTT_GLOBAL char *)dst + ((col + (s << LO)) << 3));
    u64x2 w;
    w.x = v0[s];
    w.y = v1[s];
    __builtin_nontemporal_store(w, p);
  }
}

// Column pass of EC = 6 .. 8 stages (LCOL) through LDS: a workgroup holds 2^EC
// rows of LC neighbouring columns, one column and 16 rows per lane.  The four
// stages of the largest gaps and the EC - 4 others are two register rounds
// with one LDS exchange between them; words of a row lie side by side in LDS
// as in memory, so that no access conflicts.  The first round's twiddles are
// scalar loads, and with 64 columns the second's too (a wave then holds one
// set of rows).  ld(row) and st(row, word) move this lane's word.
//
// Passes of five stages in registers alone run at the rate of a copy with the
// VALU half idle, while the fused product and key-switch blocks behind them
// are bound by VALU issue: every stage moved here takes seven (tensor) or
// three (polymul) transforms' worth of instructions from those.  64 columns
// for 6 and 7 stages, 16 for 8: at 7 stages 32 columns (half the workgroup)
// were 2-4% slower on the tensors, at 8 stages 64 columns (1024 lanes, one
// workgroup per CU) 5%.
template <int EC> constexpr uint32_t LC = EC == 8 ? 16u : 64u;
// This lane's first row group: rows (r << (EC - 4)) + w, r < 16, in the round of
// the large gaps, rows (w G + g << (EC - 4)) + k in the other.
template <int EC> __device__ __forceinline__ uint32_t lcol_w() {
  const uint32_t w = threadIdx.x / LC<EC>;
  if constexpr (LC<EC> == 64) return __builtin_amdgcn_readfirstlane(w);
  else return w;
}
// Forward stages of the words v (row map of the large gaps).
template <int LOGN, int EC, bool FIX, typename STO>
__device__ __forceinline__ void lcol_fwd(uint64_t (&v)[16], STO st, const TwM *t, const NttConst &c, uint64_t *lds) {
  constexpr int R1 = 4, R2 = EC - R1, G = 16 >> R2;
  static_assert(R2 >= 2 && R2 <= 4, "two rounds of at most 16 words");
  const uint32_t w = lcol_w<EC>();
  uint64_t *l = lds + threadIdx.x % LC<EC>;
  uint64_t a[G][1 << R2];
  fwd_round<LOGN, R1, LOGN - R1, R1, FIX>(v, LOGN, 0, 0, t, c);
#pragma unroll
  for (uint32_t r = 0; r < 16; ++r) l[((r << R2) + w) * LC<EC>] = v[r];
  __syncthreads();
#pragma unroll
  for (uint32_t g = 0; g < G; ++g) {
    const uint32_t hi = w * G + g;
#pragma unroll
    for (uint32_t k = 0; k < (1u << R2); ++k) a[g][k] = l[((hi << R2) + k) * LC<EC>];
  }
#pragma unroll
  for (uint32_t g = 0; g < G; ++g) {
    const uint32_t hi = w * G + g;
    fwd_round<LOGN, R2, LOGN - EC, R2, FIX>(a[g], LOGN, hi << (LOGN - R1), 0, t, c);
#pragma unroll
    for (uint32_t k = 0; k < (1u << R2); ++k) st((hi << R2) + k, a[g][k]);
  }
}
// Inverse stages into v (row map of the large gaps), canonical words.
template <int LOGN, int EC, bool FIX, typename LD>
__device__ __forceinline__ void lcol_inv(uint64_t (&v)[16], LD ld, const TwM *t, const NttConst &c, uint64_t *lds) {
  constexpr int R1 = 4, R2 = EC - R1, G = 16 >> R2;
  static_assert(R2 >= 2 && R2 <= 4, "two rounds of at most 16 words");
  const uint32_t w = lcol_w<EC>();
  uint64_t *l = lds + threadIdx.x % LC<EC>;
  uint64_t a[G][1 << R2];
#pragma unroll
  for (uint32_t g = 0; g < G; ++g) {
#pragma unroll
    for (uint32_t k = 0; k < (1u << R2); ++k) a[g][k] = ld(((w * G + g) << R2) + k);
  }
#pragma unroll
  for (uint32_t g = 0; g < G; ++g) {
    const uint32_t hi = w * G + g;
    inv_round<LOGN, R2, LOGN - EC, R2, LB_PASS, LB_ROUND, FIX>(a[g], LOGN, hi << (LOGN - R1), 0, t, c);
#pragma unroll
    for (uint32_t k = 0; k < (1u << R2); ++k) l[((hi << R2) + k) * LC<EC>] = a[g][k];
  }
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < 16; ++r) v[r] = l[((r << R2) + w) * LC<EC>];
  inv_round<LOGN, R1, LOGN - R1, R1, LB_ROUND, LB_PASS, FIX>(v, LOGN, 0, 0, t, c);
  reduce_out<R1, FIX>(v, c);
}
template <int LOGN, int EC, bool INV, bool FIX, typename LD, typename STO>
__device__ __forceinline__ void lcol_pass(LD ld, STO st, const TwM *t, const NttConst &c, uint64_t *lds) {
  uint64_t v[16];
  const uint32_t w = lcol_w<EC>();
  if constexpr (!INV) {
#pragma unroll
    for (uint32_t r = 0; r < 16; ++r) v[r] = ld((r << (EC - 4)) + w);
    lcol_fwd<LOGN, EC, FIX>(v, st, t, c, lds);
  } else {
    lcol_inv<LOGN, EC, FIX>(v, ld, t, c, lds);
#pragma unroll
    for (uint32_t r = 0; r < 16; ++r) st((r << (EC - 4)) + w, v[r]);
  }
}

// Geometry of a column pass of EC stages: lanes and LDS words of a workgroup,
// workgroups per polynomial.
template <int EC> constexpr bool LCOL = EC >= 6;
template <int EC> constexpr uint32_t cols_lds() { return LCOL<EC> ? LC<EC> << EC : 2u; }
template <int EC> constexpr uint32_t cols_lanes() { return LCOL<EC> ? (LC<EC> << EC) / 16 : 256u; }
template <int LOGN, int EC> constexpr uint32_t cols_blocks_per_unit() {
  return LCOL<EC> ? (1u << (LOGN - EC)) / LC<EC> : (1u << (LOGN - EC)) / (256 * ColCpl<EC>::value);
}

// Workgroup `blk` of a column pass over batch x limbs units of every
// component of `a` (the body of k_cols and of its grouped form).
template <int LOGN, int E, bool INV>
__device__ __forceinline__ void cols_block(const ColArgs &a, const TwM *__restrict__ tw,
                                           const NttConst *__restrict__ lc, uint32_t batch, uint32_t limbs,
                                           uint32_t blk) {
  __shared__ uint64_t lds[cols_lds<E>()];
  constexpr uint32_t CPL = ColCpl<E>::value;
  constexpr uint32_t tiles = cols_blocks_per_unit<LOGN, E>();
  const uint32_t units = batch * limbs;
  const uint32_t tile = blk % tiles;
  const uint32_t r = blk / tiles;
  const uint32_t comp = r / units, u = r % units;
  const uint32_t limb = u / batch, b = u % batch;
  const NttConst c = lc[limb];
  const uint64_t off = (uint64_t)limb << LOGN;
  const uint64_t *src = a.src[comp] + (uint64_t)b * a.src_sb + off;
  uint64_t *dst = a.dst[comp] + (uint64_t)b * a.dst_sb + off;
  const TwM *t = tw + ((size_t)limb * 2 + (INV ? 1 : 0)) * (1u << LOGN);
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    constexpr bool FIX = decltype(FX)::value;
    if constexpr (LCOL<E>) {
      const uint32_t col = tile * LC<E> + threadIdx.x % LC<E>;
      lcol_pass<LOGN, E, INV, FIX>([&](uint32_t row) { return gload<true>(src, (row << (LOGN - E)) + col); },
                                   [&](uint32_t row, uint64_t v) { gstore<true>(dst, (row << (LOGN - E)) + col, v); },
                                   t, c, lds);
    } else if constexpr (CPL == 2) {
      col_pass2<LOGN, E, INV, FIX>(src, dst, tile * 512 + 2 * threadIdx.x, t, c);
    } else {
      col_pass<LOGN, E, INV, FIX>(src, dst, tile * 256 + threadIdx.x, t, c);
    }
  });
}

template <int LOGN, int E, bool INV>
__global__ __launch_bounds__(cols_lanes<E>()) void k_cols(ColArgs a, const TwM *__restrict__ tw,
                                                          const NttConst *__restrict__ lc, uint32_t batch,
                                                          uint32_t limbs) {
  cols_block<LOGN, E, INV>(a, tw, lc, batch, limbs, blockIdx.x);
}

// Block pass of the forward transform: the last ST stages, on 2^(B - ST)
// contiguous blocks of 2^ST elements per workgroup; canonical output.
template <int LOGN, int ST, int B, int E>
__global__ __launch_bounds__(1 << (B - E)) void k_fwd_blocks(uint64_t *__restrict__ x, const TwM *__restrict__ tw,
                                                              const NttConst *__restrict__ lc, uint32_t batch,
                                                              uint32_t limbs) {
  __shared__ __attribute__((aligned(16))) uint64_t lds[LdsSize<B>::value];
  constexpr uint32_t tiles = 1u << (LOGN - B);
  const Unit un = unit_of(blockIdx.x, tiles, batch, limbs);
  const NttConst c = lc[un.limb];
  const TwM *t = tw + (size_t)un.limb * 2 * (1u << LOGN);
  const uint32_t blockStart = un.tile << B;
  uint64_t *p = x + (size_t)un.poly * (1u << LOGN) + blockStart;
  const uint32_t tid = threadIdx.x;
  using F = FwdFirst<ST, E>;
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    constexpr bool FIX = decltype(FX)::value;
    uint64_t v[1 << E];
    load_global<B, E, F::LO, F::R>(v, p, RoundMap<B, E, F::LO, F::R>::lane_part(tid));
    fwd_block_rounds<B, E, F::LO, F::R, FIX>(v, LOGN, lds, tid, blockStart, t, c);
    reduce_out<E, FIX>(v, c);
    store_global_m0<B, E>(v, p, lds, tid);
  });
}

// Block pass of the inverse transform: stages 0 .. ST-1; lazy output below 16q.
template <int LOGN, int ST, int B, int E>
__global__ __launch_bounds__(1 << (B - E)) void k_inv_blocks(InvIO io, const TwM *__restrict__ tw,
                                                              const NttConst *__restrict__ lc, uint32_t batch,
                                                              uint32_t limbs) {
  __shared__ __attribute__((aligned(16))) uint64_t lds[LdsSize<B>::value];
  constexpr uint32_t tiles = 1u << (LOGN - B);
  const Unit un = unit_of(blockIdx.x, tiles, batch, limbs);
  const NttConst c = lc[un.limb];
  const TwM *it = tw + ((size_t)un.limb * 2 + 1) * (1u << LOGN);
  const uint32_t blockStart = un.tile << B;
  const uint64_t *src = io.src + un.b * io.src_sb + ((uint64_t)un.limb << LOGN) + blockStart;
  uint64_t *dst = io.dst + un.b * io.dst_sb + ((uint64_t)un.limb << LOGN) + blockStart;
  const uint32_t tid = threadIdx.x;
  using L = InvLast<ST, E>;
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    constexpr bool FIX = decltype(FX)::value;
    uint64_t v[1 << E];
    load_global_m0_fresh<B, E>(v, src, lds, tid);
    inv_block_rounds<B, ST, E, 0, E, FIX>(v, LOGN, lds, tid, blockStart, it, c);
    store_global<B, E, L::LO, L::R>(v, dst, RoundMap<B, E, L::LO, L::R>::lane_part(tid));
  });
}

// ------------------------------------------------------ fused products ----
// Products of section II: PROD_MUL is the dyadic product of two polynomials
// (a (.) b); PROD_TENSOR the ciphertext Mul tensor (c0 d0, c0 d1 + c1 d0,
// c1 d1) with the middle term reduced once (mad_mod, section III-A-1).
enum { PROD_MUL = 0, PROD_TENSOR = 1 };
template <int MODE> struct ProdShape {
  static constexpr int NIN = MODE == PROD_MUL ? 2 : 4;
  static constexpr int NOUT = MODE == PROD_MUL ? 1 : 3;
};
struct ProdArgs {
  const uint64_t *in[4];
  uint64_t *out[3];
  uint64_t in_sb, out_sb;  // words between consecutive batch entries
};

// arr[i] for a wave-uniform i < N, as a chain of selects: indexing the
// kernel-argument array with a loop counter directly made the compiler copy
// it to scratch and load the pointer from there into VGPRs.
// Each element passes through an (empty) scalar-register asm first, so the
// select chain is not folded back into an indexed load.
template <typename T, int N> __device__ __forceinline__ T pick_ptr(T const (&arr)[N], int i) {
  T r = arr[0];
  asm volatile("" : "+s"(r));
#pragma unroll
  for (int k = 1; k < N; ++k) {
    T c = arr[k];
    asm volatile("" : "+s"(c));
    r = (i == k) ? c : r;
  }
  return r;
}

template <int MODE, int E>
__device__ __forceinline__ void products(uint64_t (&X)[ProdShape<MODE>::NIN][1 << E],
                                         uint64_t (&Y)[ProdShape<MODE>::NOUT][1 << E], const NttConst &c) {
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) {
    if constexpr (MODE == PROD_MUL) {
      Y[0][s] = mulmod(X[0][s], X[1][s], c.q, c.mu, c.k);
    } else {
      Y[0][s] = mulmod(X[0][s], X[2][s], c.q, c.mu, c.k);
      Y[1][s] = madmod(X[0][s], X[3][s], X[1][s], X[2][s], c.q, c.mu, c.k);
      Y[2][s] = mulmod(X[1][s], X[3][s], c.q, c.mu, c.k);
    }
  }
}

// The products ahead of an inverse transform: every output is off by a constant
// factor, which the inverse transform removes with its N^-1 scaling, taken from
// the folded constants.
//   34..55 bits (not FIX)  mont30_mul, off by 2^-60; factors below 3q, outputs
//                below 6q.  N = 2^16, 24 primes, 32 ciphertext pairs: 960 us of
//                product kernel, 1000 with the form below.
//   others       Montgomery products with R = 2^64; MUL factors below 4q
//                (a b < 16 q^2 < q R as q < 2^60), TENSOR factors below 2q
//                (c0 d1 + c1 d0 < 8 q^2 < q R), outputs in [0, 2q).  By
//                mont30_mul, with one factor cut below q and the result below
//                3q, the registers grow: 1% slower (2^15, 16 primes of 50 to 60
//                bits, 128 products) and, the tensor at three waves for four or
//                spilling, 5% even where no such modulus occurs.
template <int MODE, int E, bool FIX>
__device__ __forceinline__ void products_mont(uint64_t (&X)[ProdShape<MODE>::NIN][1 << E],
                                              uint64_t (&Y)[ProdShape<MODE>::NOUT][1 << E], const NttConst &c,
                                              uint64_t qinv) {
  const uint32_t four = opaque4();
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) {
    if constexpr (FIX && MODE == PROD_MUL) {
      Y[0][s] = mont_mul(X[0][s], X[1][s], c.q, qinv);
    } else if constexpr (FIX) {
      Y[0][s] = mont_mul(X[0][s], X[2][s], c.q, qinv);
      Y[1][s] = mont_mad(X[0][s], X[3][s], X[1][s], X[2][s], c.q, qinv);
      Y[2][s] = mont_mul(X[1][s], X[3][s], c.q, qinv);
    } else if constexpr (MODE == PROD_MUL) {
      Y[0][s] = mont30_mul(split30(X[0][s]), X[1][s], c, four);
    } else {
      const Split30 a0 = split30(X[0][s]), a1 = split30(X[1][s]);
      Y[0][s] = mont30_mul(a0, X[2][s], c, four);
      Y[1][s] = mont30_mad(a0, X[3][s], a1, X[2][s], c, four);
      Y[2][s] = mont30_mul(a1, X[3][s], c, four);
    }
  }
}

// Forward outputs brought to the factor ranges of the products: lazy words of 34
// to 55 bits (below 256q) below 3q, of 56 bits and more below 2q, of 33 bits and
// fewer (below 207q: 17 stages of 12q on inputs below 3q) as they are, which keeps
// the tensor's sum of two products below q R (2 (207 q)^2 < q 2^64).
template <int E, bool FIX> __device__ __forceinline__ void reduce_for_mont(uint64_t (&x)[1 << E], const NttConst &c) {
#pragma unroll
  for (int s = 0; s < (1 << E); ++s) {
    if constexpr (!FIX) x[s] = est3(x[s], c);
    else if (c.k >= 34) x[s] = reduce_est(x[s], c.nq, c.ce, c.k - 33);
  }
}

// One workgroup per block of 2^B coefficients of one (batch entry, limb):
// forward block rounds of every input (DO_FWD; otherwise the inputs are
// already NTT-domain values), the products in registers, then the inverse
// block rounds of every output (DO_INV).  The forward transform ends and the
// inverse transform begins with each lane holding 2^E consecutive NTT-domain
// values, so the product needs no data exchange and the NTT-domain values
// never leave the chip.  With B == LOGN the whole product is one kernel;
// with B < LOGN the forward column pass runs before it and the inverse
// column pass after it.  With DO_INV the products are Montgomery products
// and lc must hold the folded constants (N^-1 scaled), also for
// the inverse column pass that completes the transform.  Without DO_INV the
// products are exact (Barrett) and lc the plain constants.
template <int LOGN, int ST, int B, int E, int MODE, bool DO_FWD, bool DO_INV, bool FIX>
__device__ __forceinline__ void prod_body(const ProdArgs &a, uint64_t in_off, uint64_t out_off, uint32_t blockStart,
                                          const TwM *t, const NttConst &c, const MontLimb *mont, uint64_t *lds) {
  constexpr int NIN = ProdShape<MODE>::NIN, NOUT = ProdShape<MODE>::NOUT;
  constexpr bool PRE = MODE == PROD_MUL && LOGN > 9;  // see fwd_block_rounds
  const TwM *it = t + (1u << LOGN);
  const uint32_t tid = threadIdx.x;
  using F = FwdFirst<ST, E>;
  using L = InvLast<ST, E>;
  // The transform code appears once for all inputs and once for all outputs
  // (rolled loops): unrolled per polynomial it would outgrow the instruction
  // cache.  Results move between the loop's working registers and the
  // per-polynomial arrays through compile-time-indexed copies.
  uint64_t X[NIN][1 << E];
#pragma unroll 1
  for (int p = 0; p < NIN; ++p) {
    uint64_t v[1 << E];
    if constexpr (DO_FWD) {
      if (p > 0) __syncthreads();  // the previous input's last LDS reads are done
      // an opaque copy of the table pointer per input: the twiddles are re-read
      // from cache instead of being hoisted out of the loop into VGPRs
      const TwM *tp = opaque(t);
      load_global<B, E, F::LO, F::R, true>(v, pick_ptr(a.in, p) + in_off, RoundMap<B, E, F::LO, F::R>::lane_part(tid));
      fwd_block_rounds<B, E, F::LO, F::R, FIX, PRE>(v, LOGN, lds, tid, blockStart, tp, c);
      if constexpr (DO_INV) reduce_for_mont<E, FIX>(v, c);
      else reduce_out<E, FIX>(v, c);
    } else {
      load_global_m0<B, E, true>(v, pick_ptr(a.in, p) + in_off, lds, tid);
    }
    static_for<0, NIN>([&](auto P) {
      if (p == decltype(P)::value) {
        // distinct marker per branch: keeps the branches from being merged
        // into one dynamically indexed (stack) store
        if constexpr (MODE == PROD_TENSOR) asm volatile("; sel %0" ::"n"(decltype(P)::value));
#pragma unroll
        for (int s2 = 0; s2 < (1 << E); ++s2) X[decltype(P)::value][s2] = v[s2];
      }
    });
  }
  uint64_t Y[NOUT][1 << E];
  if constexpr (DO_INV) products_mont<MODE, E, FIX>(X, Y, c, mont->qinv);
  else products<MODE, E>(X, Y, c);
#pragma unroll 1
  for (int o = 0; o < NOUT; ++o) {
    uint64_t v[1 << E];
    static_for<0, NOUT>([&](auto O) {
      if (o == decltype(O)::value) {
        if constexpr (MODE == PROD_TENSOR) asm volatile("; sel %0" ::"n"(decltype(O)::value));
#pragma unroll
        for (int s2 = 0; s2 < (1 << E); ++s2) v[s2] = Y[decltype(O)::value][s2];
      }
    });
    if constexpr (DO_INV) {
      __syncthreads();  // earlier LDS reads of this workgroup are done
      inv_block_rounds<B, ST, E, 0, E, FIX, PRE>(v, LOGN, lds, tid, blockStart, opaque(it), c);
      if constexpr (ST == LOGN) reduce_out<E, FIX>(v, c);
      store_global<B, E, L::LO, L::R>(v, pick_ptr(a.out, o) + out_off, RoundMap<B, E, L::LO, L::R>::lane_part(tid));
    } else {
      store_global_m0<B, E>(v, pick_ptr(a.out, o) + out_off, lds, tid);
    }
  }
}

// Workgroup `blk` of the fused product over batch x limbs units (the body of
// k_prod and of its grouped form).
template <int LOGN, int ST, int B, int E, int MODE, bool DO_FWD, bool DO_INV>
__device__ __forceinline__ void prod_block(const ProdArgs &a, const TwM *__restrict__ tw,
                                           const NttConst *__restrict__ lc, const MontLimb *__restrict__ mont,
                                           uint32_t batch, uint32_t limbs, uint32_t blk) {
  __shared__ __attribute__((aligned(16))) uint64_t lds[(DO_FWD || DO_INV) ? LdsSize<B>::value : 2];
  constexpr uint32_t tiles = 1u << (LOGN - B);
  const uint32_t tile = blk % tiles;
  const uint32_t r = blk / tiles;
  const uint32_t limb = r / batch, b = r % batch;
  const NttConst c = lc[limb];
  const TwM *t = tw + (size_t)limb * 2 * (1u << LOGN);
  const uint32_t blockStart = tile << B;
  const uint64_t in_off = (uint64_t)b * a.in_sb + ((uint64_t)limb << LOGN) + blockStart;
  const uint64_t out_off = (uint64_t)b * a.out_sb + ((uint64_t)limb << LOGN) + blockStart;
  by_class(c, [&](auto FX) __attribute__((always_inline)) {
    prod_body<LOGN, ST, B, E, MODE, DO_FWD, DO_INV, decltype(FX)::value>(a, in_off, out_off, blockStart, t, c, mont + limb,
                                                                     lds);
  });
}

// Waves per SIMD asked of the compiler.  The tensor of NTT-domain inputs with
// coefficient-domain outputs takes 130 to 133 VGPRs at 2^11 and 2^12 by itself, which
// at 2^12 leaves one workgroup of 8 waves per CU; held to 128, two (2^12, 4096 units:
// 379 -> 297 us, 463 -> 339 with 60-bit moduli; 2^11 167 -> 152 with those).
constexpr int prod_waves(int e, int mode, bool do_fwd, bool do_inv) {
  return mode == PROD_TENSOR && !do_fwd && do_inv && e == 3 ? 4 : 1;
}

template <int LOGN, int ST, int B, int E, int MODE, bool DO_FWD, bool DO_INV>
__global__ __launch_bounds__(1 << (B - E), prod_waves(E, MODE, DO_FWD, DO_INV)) void k_prod(ProdArgs a, const TwM *__restrict__ tw,
                                                        const NttConst *__restrict__ lc,
                                                        const MontLimb *__restrict__ mont, uint32_t batch,
                                                        uint32_t limbs) {
  prod_block<LOGN, ST, B, E, MODE, DO_FWD, DO_INV>(a, tw, lc, mont, batch, limbs, blockIdx.x);
}

// Element-wise products of NTT-domain inputs (no transform): tiles of 2048
// words of one (batch entry, limb), coalesced, limb constants uniform per
// workgroup.
template <int MODE>
__device__ __forceinline__ void elem_block(const ProdArgs &a, const NttConst *__restrict__ lc, uint32_t batch,
                                           uint32_t limbs, uint32_t log_n, uint32_t tiles, uint32_t blk) {
  constexpr int NIN = ProdShape<MODE>::NIN, NOUT = ProdShape<MODE>::NOUT;
  const uint32_t tile = blk % tiles;
  const uint32_t r = blk / tiles;
  const uint32_t limb = r / batch, b = r % batch;
  const NttConst c = lc[limb];
  const uint32_t n = 1u << log_n;
  const uint64_t in_off = (uint64_t)b * a.in_sb + ((uint64_t)limb << log_n) + tile * 2048u;
  const uint64_t out_off = (uint64_t)b * a.out_sb + ((uint64_t)limb << log_n) + tile * 2048u;
  uint64_t X[NIN][8], Y[NOUT][8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const uint32_t i = threadIdx.x + 256u * s;
#pragma unroll
    for (int p = 0; p < NIN; ++p) X[p][s] = (tile * 2048u + i < n) ? a.in[p][in_off + i] : 0;
  }
  products<MODE, 3>(X, Y, c);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const uint32_t i = threadIdx.x + 256u * s;
    if (tile * 2048u + i < n) {
#pragma unroll
      for (int o = 0; o < NOUT; ++o) a.out[o][out_off + i] = Y[o][s];
    }
  }
}

template <int MODE>
__global__ __launch_bounds__(256) void k_elem(ProdArgs a, const NttConst *__restrict__ lc, uint32_t batch,
                                              uint32_t limbs, uint32_t log_n, uint32_t tiles) {
  elem_block<MODE>(a, lc, batch, limbs, log_n, tiles, blockIdx.x);
}

}  // namespace hentt
