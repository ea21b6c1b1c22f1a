// Plain records shared by the device kernels and the host-side table builder
// (no HIP dependencies, so the host code that fills them can be built and
// tested by a plain C++ compiler).
#pragma once
#include <stdint.h>

namespace hentt {

// Moduli constants used by the butterflies.
struct ModQ {
  uint64_t q, nq, q2, nq2, q4, nq4;  // q, 2q, 4q and their negations mod 2^64
};

struct LimbConst {
  ModQ m;                   // q, 2q, 4q and their negations mod 2^64
  uint64_t ninv, ninv_s;    // N^-1 mod q and its Shoup quotient
  uint64_t ninvw, ninvw_s;  // N^-1 * psi^-brv(1) mod q and its Shoup quotient
  uint64_t mu;              // floor(2^(2k) / q), k = bit length of q (Barrett)
  uint32_t k, pad;
};

static_assert(sizeof(LimbConst) == 96, "limb records are 12 words (documented in the C ABI)");

// Montgomery constants of a limb (R = 2^64).
struct MontLimb {
  uint64_t qinv;   // -q^-1 mod 2^64
  uint64_t r, rs;  // R mod q and its Shoup quotient
  uint64_t pad;
};

// A root power in the form the transforms multiply by (mul_tw in modarith.hpp):
// A = W 2^30 mod q and B = W 2^62 mod q, each split at bit 30 (A = a1 2^30 + a0,
// B = b1 2^30 + b0), in one 16-byte word.
struct alignas(16) TwM { uint32_t a0, a1, b0, b1; };

// Per-limb constants of the transforms.
struct alignas(16) NttConst {
  uint64_t q, nq;        // q and -q mod 2^64
  uint64_t mu;           // floor(2^(2k) / q) (Barrett)
  uint64_t off;          // 12 q, the bound of a mul_tw product
  uint32_t qlo, qhi;     // q split at bit 30
  uint32_t qi;           // -qlo^-1 mod 2^32
  uint32_t k;            // bit length of q
  uint32_t c64;          // floor(2^64 / q) (k >= 34, else 0)
  uint32_t ce;           // floor(2^(k+31) / q)
  uint32_t s0, s1;       // shifts of the quotient estimate of reduce_word
  TwM ninv, ninvw;       // N^-1 and N^-1 psi^-brv(1)
};
static_assert(sizeof(NttConst) == 96, "read field by field as 12 words (ld_nc)");

// 2^30 mod q and 2^62 mod q as root powers: they bring a plain word into TwM form
// (the matrix product).
struct MatLimb { TwM w30, w62; };

// A root power and its Shoup quotient (W, W' = floor(W 2^64 / q)), Algorithm 1.
struct alignas(16) Tw { uint64_t w, ws; };

}  // namespace hentt
