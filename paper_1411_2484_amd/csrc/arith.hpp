// Device arithmetic for gfx950: Montgomery products over 32-bit words (and
// 64-bit moduli from 32-bit limbs), Mersenne reductions for the skip
// generators, and the wave-level helpers the kernels use.
//
// A 32 x 32 -> 64 product (plus a 64-bit addend) is one v_mad_u64_u32; on
// gfx950 it issues at about 60% of the rate of a plain 32-bit add, so the
// 64-bit routines below are arranged to need few of them and few carries
// (the one carry the Montgomery reduction cannot avoid is the
// multiply-add's own carry-out).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "layout.hpp"

namespace phprng {

// Clears the calling thread's last HIP error before a launch whose error is
// read with hipGetLastError: a call that failed earlier in the process (an
// allocation refused somewhere else, say) would otherwise be reported as
// this launch's failure.
inline void clear_launch_error() { (void)hipGetLastError(); }

namespace dev {

// ---- skip generator mod 2^31 - 1 (eq. (5), width 32) ----------------------

// One skip step left unreduced: v' = a v mod p up to one subtraction of p,
// for v < 2^32 nonzero mod p.  With the doubled multiplier the product's high
// word is (a v) >> 31 and its low word is twice (a v) mod 2^31, so the
// Mersenne fold needs no mask and no funnel shift.  v' = (low half) + (high
// word) <= p + 2a < 2p, and v' is never 0 or p.
__device__ __forceinline__ uint32_t step_p31(uint32_t v) {
  static_assert(2ull * kA32 < kP32, "the doubled multiplier keeps v' below 2p");
  const uint64_t t = (uint64_t)v * (2u * kA32);
  return ((uint32_t)t >> 1) + (uint32_t)(t >> 32);
}

// v mod p for v < 2p, v != p: subtract p once when v > p.
__device__ __forceinline__ uint32_t fold_p31(uint32_t v) { return min(v, v - kP32); }

// x y mod (2^31 - 1) for x, y in [1, 2^31 - 2] (the same fold, y doubled here).
__device__ __forceinline__ uint32_t mulmod_p31(uint32_t x, uint32_t y) {
  const uint64_t t = (uint64_t)x * (y + y);
  return fold_p31(((uint32_t)t >> 1) + (uint32_t)(t >> 32));
}

__device__ __forceinline__ uint32_t powmod_p31(uint32_t b, uint64_t e) {
  uint32_t r = 1;
  while (e) {
    if (e & 1) r = mulmod_p31(r, b);
    b = mulmod_p31(b, b);
    e >>= 1;
  }
  return r;
}

// One in an SGPR that the compiler cannot fold to a constant.
__device__ __forceinline__ uint32_t opaque_one() {
  uint32_t one;
  asm volatile("s_mov_b32 %0, 1" : "=s"(one));
  return one;
}

// acc + x as a single v_mad_u64_u32 (x * one + acc, one == 1): the 32-bit
// addend needs no zero-extended register pair.
__device__ __forceinline__ uint64_t acc_u32(uint64_t acc, uint32_t x, uint32_t one) {
  return (uint64_t)x * one + acc;
}

// ---- 32-bit Montgomery arithmetic modulo n in [2^31, 2^32) ----------------

// x y 2^{-32} mod n for x, y < n; ninv = n^{-1} mod 2^32.  The low words of
// x y and q n cancel exactly, so the result is hi(x y) - hi(q n) (+ n).
// Six VALU instructions: v_mad_u64_u32, v_mul_lo_u32, v_mul_hi_u32,
// v_sub_co_u32 (borrow), v_cndmask_b32, v_add_u32.
__device__ __forceinline__ uint32_t mont32(uint32_t x, uint32_t y, uint32_t n, uint32_t ninv) {
  uint64_t t = (uint64_t)x * y;
  uint32_t q = (uint32_t)t * ninv;
  uint32_t qh = __umulhi(q, n);
  uint32_t r;
  bool borrow = __builtin_usub_overflow((uint32_t)(t >> 32), qh, &r);
  return r + (borrow ? n : 0u);
}

// +-(x^2 2^{-32}) mod n for x <= n: the absolute value of the difference that
// mont32 corrects by n.  The next squaring does not see the sign, and one
// v_sad_u32 replaces the borrow, the select and the add (4 instructions
// instead of 6, 4.1 instead of 5.3 issue cycles).
__device__ __forceinline__ uint32_t msqr32_abs(uint32_t x, uint32_t n, uint32_t ninv) {
  const uint64_t t = (uint64_t)x * x;
  const uint32_t q = (uint32_t)t * ninv;
  const uint32_t qh = __umulhi(q, n);
  uint32_t r;
  asm("v_sad_u32 %0, %1, %2, 0" : "=v"(r) : "v"((uint32_t)(t >> 32)), "v"(qh));
  return r;
}

// v 2^{-32} mod n for v < n 2^32.
__device__ __forceinline__ uint32_t redc32(uint64_t v, uint32_t n, uint32_t ninv) {
  uint32_t q = (uint32_t)v * ninv;
  uint32_t qh = __umulhi(q, n);
  uint32_t r;
  bool borrow = __builtin_usub_overflow((uint32_t)(v >> 32), qh, &r);
  return r + (borrow ? n : 0u);
}

// (m + s) mod n for m, s < n.
__device__ __forceinline__ uint32_t addmod32(uint32_t m, uint32_t s, uint32_t n) {
  uint32_t ns = n - s;
  uint32_t d = m - ns;
  return m < ns ? d + n : d;
}

// (w - s) mod n for w <= n, 1 <= s < n: the borrow selects the n added back
// (one instruction less than the sum).
__device__ __forceinline__ uint32_t submod32(uint32_t w, uint32_t s, uint32_t n) {
  uint32_t r;
  const bool borrow = __builtin_usub_overflow(w, s, &r);
  return r + (borrow ? n : 0u);
}

// x^e mod n (plus PLUS, 0 or 1) by left-to-right square-and-multiply on the
// unconverted x <= n, e odd: the chain yields x^e 2^{-32(e-1)}, and one
// product with kc = 2^{32 e} mod n removes the factor.  With kc =
// -2^{32 e} mod n and x = n - m it returns m^e (e is odd).  Squarings that
// feed another squaring keep only the absolute value.  EK selects a fixed
// chain (3, 5, 9, 17) or 0 for a chain over the bits of e.
template <int EK, int PLUS = 0>
__device__ __forceinline__ uint32_t encrypt32(uint32_t m, uint32_t n, uint32_t ninv, uint32_t kc, uint64_t e,
                                              int ebits) {
  uint32_t x = m;
  if constexpr (EK == 5) {
    x = msqr32_abs(x, n, ninv);
  } else if constexpr (EK == 9) {
    x = msqr32_abs(x, n, ninv);
    x = msqr32_abs(x, n, ninv);
  } else if constexpr (EK == 17) {
    x = msqr32_abs(x, n, ninv);
    x = msqr32_abs(x, n, ninv);
    x = msqr32_abs(x, n, ninv);
  }
  if constexpr (EK != 0) {
    x = mont32(x, x, n, ninv);
    x = mont32(x, m, n, ninv);
  } else {
    for (int b = ebits - 2; b >= 0; --b) {
      if ((e >> b) & 1)
        x = mont32(mont32(x, x, n, ninv), m, n, ninv);
      else
        x = msqr32_abs(x, n, ninv);
    }
  }
  // the last product, with PLUS in the two values that the borrow selects
  const uint64_t t = (uint64_t)x * kc;
  const uint32_t q = (uint32_t)t * ninv;
  const uint32_t qh = __umulhi(q, n);
  uint32_t r;
  const bool borrow = __builtin_usub_overflow((uint32_t)(t >> 32), qh, &r);
  return r + (borrow ? n + PLUS : (uint32_t)PLUS);
}

// a / den correctly rounded for integers 1 <= a < den <= 2^33, with rcp =
// RN(1/den) and rcp_lo = RN(1/den - rcp): a rcp + RN(a rcp_lo) is within
// 2^-105 of a/den (relative) and the fma rounds it once, while no rounding
// boundary of binary64 comes closer to a/den than 2^-88 (ulp/2^34).
__device__ __forceinline__ double uniform32(uint32_t c1, double rcp, double rcp_lo) {
  const double a = (double)c1;
  return __builtin_fma(a, rcp, a * rcp_lo);
}

// ---- 64-bit moduli from 32-bit limbs --------------------------------------

struct W128 {
  uint64_t lo, hi;
};

// a b + c in one v_mad_u64_u32.  Written out because the compiler
// reassociates a sum of two such products plus a 32-bit term into two
// products and a separate 64-bit add.
__device__ __forceinline__ uint64_t mad_u64_u32(uint32_t a, uint32_t b, uint64_t c) {
  uint64_t r, carry;
  asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(r), "=s"(carry) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Full product of x, y < 2^63.  The high words are below 2^31, so
// x1 y0 + x0 y1 + hi(x0 y0) < 2^64: three multiply-adds chain without a
// carry, and each 64-bit addend is a whole register pair.
__device__ __forceinline__ W128 mul63w(uint64_t x, uint64_t y) {
  const uint32_t x0 = (uint32_t)x, x1 = (uint32_t)(x >> 32);
  const uint32_t y0 = (uint32_t)y, y1 = (uint32_t)(y >> 32);
  const uint64_t p00 = (uint64_t)x0 * y0;
  const uint64_t mid = mad_u64_u32(x1, y0, (uint64_t)x0 * y1 + (p00 >> 32));
  return {(mid << 32) | (uint32_t)p00, (uint64_t)x1 * y1 + (mid >> 32)};
}

// High word of q n for n < 2^63: with h = hi(q0 n0), a = q1 n0 + h < 2^64
// and b = q0 n1 + lo(a) < 2^64, the high word is q1 n1 + hi(a) + hi(b).
__device__ __forceinline__ uint64_t mulhi_n63(uint64_t q, uint64_t n) {
  const uint32_t q0 = (uint32_t)q, q1 = (uint32_t)(q >> 32);
  const uint32_t n0 = (uint32_t)n, n1 = (uint32_t)(n >> 32);
  const uint64_t a = (uint64_t)q1 * n0 + __umulhi(q0, n0);
  const uint64_t b = (uint64_t)q0 * n1 + (uint32_t)a;
  return (uint64_t)q1 * n1 + (a >> 32) + (b >> 32);
}

// v 2^{-64} mod n for v < n 2^64, n < 2^63 odd; ninv = n^{-1} mod 2^64.  The
// low words of v and q n cancel exactly, so the result is hi(v) - hi(q n)
// (+ n).
__device__ __forceinline__ uint64_t redc64(W128 v, uint64_t n, uint64_t ninv) {
  const uint64_t q = v.lo * ninv;
  const uint64_t qh = mulhi_n63(q, n);
  unsigned long r;
  bool borrow = __builtin_usubl_overflow(v.hi, qh, &r);
  return (uint64_t)r + (borrow ? n : 0ull);
}

// x y 2^{-64} mod n for x, y < n < 2^63.
__device__ __forceinline__ uint64_t mont64(uint64_t x, uint64_t y, uint64_t n, uint64_t ninv) {
  return redc64(mul63w(x, y), n, ninv);
}

// redc64 for a modulus that is the same in every lane of the wave (n and
// ninv are read from scalar registers; the compiler reads them from the
// first active lane if they sit in vector registers).  Same result as
// redc64, in fewer instructions: with q = lo(v) ninv mod 2^64 and
// h = hi(q0 n0), the middle column q1 n0 + h + q0 n1 can exceed 64 bits,
// and the multiply-add's carry-out supplies that bit, so
// hi(q n) = q1 n1 + (hi(middle) + carry 2^32) takes one multiply-add; the
// borrow of hi(v) - hi(q n) then selects the n that is added back (the
// compiler's form recomputes that borrow with a 64-bit compare).
//
// v0-v3 hold the intermediate register pairs (declared clobbered), and VCC
// carries each carry or borrow: gfx950 wants two wait states between a
// VALU write of VCC and a VALU read of it, hence the s_nop lines.
__device__ __forceinline__ uint64_t redc64_uniform(W128 v, uint64_t n, uint64_t ninv) {
  const uint64_t q = v.lo * ninv;
  const uint64_t h = __umulhi((uint32_t)q, (uint32_t)n);
  uint64_t r;
  asm("v_mad_u64_u32 v[0:1], vcc, %[q1], %[n0], %[h]\n\t"   // q1 n0 + h < 2^64
      "v_mad_u64_u32 v[0:1], vcc, %[q0], %[n1], v[0:1]\n\t"  // + q0 n1, carry-out in VCC
      "v_mov_b32 v2, v1\n\t"
      "s_nop 0\n\t"
      "v_cndmask_b32_e64 v3, 0, 1, vcc\n\t"                  // v[2:3] = hi(middle) + carry 2^32
      "v_mad_u64_u32 v[2:3], vcc, %[q1], %[n1], v[2:3]\n\t"  // hi(q n) < 2^64
      "v_sub_co_u32 v0, vcc, %[p0], v2\n\t"
      "s_nop 1\n\t"
      "v_subb_co_u32 v1, vcc, %[p1], v3, vcc\n\t"           // hi(v) - hi(q n), borrow in VCC
      "s_nop 1\n\t"
      "v_cndmask_b32 v2, 0, %[vn0], vcc\n\t"
      "v_cndmask_b32 v3, 0, %[vn1], vcc\n\t"
      "v_lshl_add_u64 %[r], v[0:1], 0, v[2:3]"               // + (borrow ? n : 0)
      : [r] "=v"(r)
      : [q0] "v"((uint32_t)q), [q1] "v"((uint32_t)(q >> 32)), [n0] "s"((uint32_t)n),
        [n1] "s"((uint32_t)(n >> 32)), [h] "v"(h), [p0] "v"((uint32_t)v.hi), [p1] "v"((uint32_t)(v.hi >> 32)),
        [vn0] "v"((uint32_t)n), [vn1] "v"((uint32_t)(n >> 32))
      : "v0", "v1", "v2", "v3", "vcc");
  return r;
}

__device__ __forceinline__ uint64_t mont64_uniform(uint64_t x, uint64_t y, uint64_t n, uint64_t ninv) {
  return redc64_uniform(mul63w(x, y), n, ninv);
}

// ---- the width-64 encryption chain ------------------------------------------
//
// Products x y 2^{-64} mod n in two rounds of 32 bits, added instead of
// subtracted: with n' = -n^{-1} mod 2^32, round 1 adds q n (q = lo32(x y) n')
// and round 2 q' n 2^32, which clear the two low words; the multiply-adds
// take the running sum as their 64-bit addend, so only three carry-outs and
// two register moves remain of the word bookkeeping.  Inputs below 2^63 give
// r = (x y + Q n) 2^{-64} < 2^62 + n < 2^64; between the products of a chain
// n is subtracted when bit 63 is set, which keeps r below 2^63 (a sign mask:
// no compare, no carry), and only the last product is reduced below n.  19
// VALU instructions per product with that step, about 16.1 issue cycles
// (21 and 18.4 with the 64-bit quotient of redc64_uniform); n, -n and n' are
// read from scalar registers (the same in every lane of the wave).
//
// v0-v7 hold the intermediate register pairs; VCC carries each carry-out
// (two wait states between its write and its read as a carry).
struct Mod64 {
  uint32_t n0, n1;    // n
  uint32_t np;        // -n^{-1} mod 2^32
  uint32_t nn0, nn1;  // 2^64 - n
  uint32_t one;       // 1 in a vector register
};

#define PHPRNG_ROUND1                                                                         \
  "v_mul_lo_u32 v7, v0, %[np]\n\t"                                                            \
  "v_mad_u64_u32 v[0:1], vcc, v7, %[n0], v[0:1]\n\t" /* lo32 = 0, carry in VCC */             \
  "v_mov_b32 v2, v1\n\t"                                                                      \
  "s_nop 0\n\t"                                                                               \
  "v_cndmask_b32 v3, 0, %[one], vcc\n\t"                                                      \
  "v_mad_u64_u32 v[2:3], vcc, v7, %[n1], v[2:3]\n\t"

// column 1 is in v[2:3] with its carry-out in VCC
#define PHPRNG_ROUND2                                                                         \
  "v_mul_lo_u32 v7, v2, %[np]\n\t"                                                            \
  "s_nop 0\n\t"                                                                               \
  "v_cndmask_b32 v5, 0, %[one], vcc\n\t"                                                      \
  "v_mad_u64_u32 v[2:3], vcc, v7, %[n0], v[2:3]\n\t" /* lo32 = 0, carry in VCC */             \
  "v_mov_b32 v4, v3\n\t"                                                                      \
  "s_nop 0\n\t"                                                                               \
  "v_addc_co_u32 v5, vcc, 0, v5, vcc\n\t"                                                     \
  "v_mad_u64_u32 v[4:5], vcc, v7, %[n1], v[4:5]\n\t"

#define PHPRNG_BELOW_2_63                                                                     \
  "v_ashrrev_i32 v6, 31, v5\n\t"                                                              \
  "v_and_b32 v0, %[nn0], v6\n\t"                                                              \
  "v_and_b32 v1, %[nn1], v6\n\t"                                                              \
  "v_lshl_add_u64 %[r], v[4:5], 0, v[0:1]"

#define PHPRNG_MOD_OPERANDS                                                                   \
  [n0] "s"(K.n0), [n1] "s"(K.n1), [np] "s"(K.np), [one] "v"(K.one)
#define PHPRNG_CLOBBERS "v0", "v1", "v2", "v3", "v4", "v5", "v6", "v7", "vcc"

// x^2 2^{-64} mod n, below 2^63, for x < 2^63.
__device__ __forceinline__ uint64_t lazy_sqr64(uint64_t x, const Mod64 &K) {
  uint64_t r;
  asm("v_mad_u64_u32 v[0:1], vcc, %[x0], %[x0], 0\n\t"
      "v_add_u32 v6, %[x1], %[x1]\n\t"
      PHPRNG_ROUND1
      "v_mad_u64_u32 v[2:3], vcc, %[x0], v6, v[2:3]\n\t"
      PHPRNG_ROUND2
      "v_mad_u64_u32 v[4:5], vcc, %[x1], %[x1], v[4:5]\n\t"
      PHPRNG_BELOW_2_63
      : [r] "=v"(r)
      : [x0] "v"((uint32_t)x), [x1] "v"((uint32_t)(x >> 32)), [nn0] "s"(K.nn0), [nn1] "s"(K.nn1),
        PHPRNG_MOD_OPERANDS
      : PHPRNG_CLOBBERS);
  return r;
}

// x y 2^{-64} mod n, below 2^63, for x, y < 2^63.
__device__ __forceinline__ uint64_t lazy_mul64(uint64_t x, uint64_t y, const Mod64 &K) {
  uint64_t r;
  asm("v_mad_u64_u32 v[0:1], vcc, %[x0], %[y0], 0\n\t"
      PHPRNG_ROUND1
      "v_mad_u64_u32 v[2:3], vcc, %[x0], %[y1], v[2:3]\n\t"  // below 2^64: n1, y1 < 2^31
      "v_mad_u64_u32 v[2:3], vcc, %[x1], %[y0], v[2:3]\n\t"
      PHPRNG_ROUND2
      "v_mad_u64_u32 v[4:5], vcc, %[x1], %[y1], v[4:5]\n\t"
      PHPRNG_BELOW_2_63
      : [r] "=v"(r)
      : [x0] "v"((uint32_t)x), [x1] "v"((uint32_t)(x >> 32)), [y0] "v"((uint32_t)y), [y1] "v"((uint32_t)(y >> 32)),
        [nn0] "s"(K.nn0), [nn1] "s"(K.nn1), PHPRNG_MOD_OPERANDS
      : PHPRNG_CLOBBERS);
  return r;
}

// (x k 2^{-64} mod n) + PLUS for x < 2^63 and a wave-uniform k < n: reduced
// below n by one compare that selects PLUS or PLUS - n.
template <int PLUS>
__device__ __forceinline__ uint64_t last_mul64(uint64_t x, uint64_t k, uint64_t n, const Mod64 &K) {
  uint64_t r;
  asm("v_mad_u64_u32 v[0:1], vcc, %[x0], %[y0], 0\n\t"
      PHPRNG_ROUND1
      "v_mad_u64_u32 v[2:3], vcc, %[x0], %[y1], v[2:3]\n\t"
      "v_mad_u64_u32 v[2:3], vcc, %[x1], %[y0], v[2:3]\n\t"
      PHPRNG_ROUND2
      "v_mad_u64_u32 %[r], vcc, %[x1], %[y1], v[4:5]"
      : [r] "=v"(r)
      : [x0] "v"((uint32_t)x), [x1] "v"((uint32_t)(x >> 32)), [y0] "s"((uint32_t)k), [y1] "s"((uint32_t)(k >> 32)),
        PHPRNG_MOD_OPERANDS
      : PHPRNG_CLOBBERS);
  return r + (r < n ? (uint64_t)PLUS : (uint64_t)PLUS - n);
}

#undef PHPRNG_ROUND1
#undef PHPRNG_ROUND2
#undef PHPRNG_BELOW_2_63
#undef PHPRNG_MOD_OPERANDS
#undef PHPRNG_CLOBBERS

// x^e mod n (plus PLUS, 0 or 1) for x <= n, e odd, by a fixed chain for e =
// 3, 5, 9, 17, else by left-to-right squaring; n, ninv and kc = 2^{64 e} mod
// n are the same in every lane of the wave (one instance per tile).  With kc
// = -2^{64 e} mod n and x = n - m it returns m^e.
template <int EK, int PLUS = 0>
__device__ __forceinline__ uint64_t encrypt64(uint64_t m, uint64_t n, uint64_t ninv, uint64_t kc, uint64_t e,
                                              int ebits) {
  const Mod64 K{(uint32_t)n, (uint32_t)(n >> 32), 0u - (uint32_t)ninv, (uint32_t)(0ull - n),
                (uint32_t)((0ull - n) >> 32), 1u};
  uint64_t x = m;
  if constexpr (EK != 0) {
    constexpr int kSquarings = EK == 3 ? 1 : (EK == 5 ? 2 : (EK == 9 ? 3 : 4));
    static_assert(EK == (1 << kSquarings) + 1, "fixed chains are 2^k + 1");
#pragma unroll
    for (int i = 0; i < kSquarings; ++i) x = lazy_sqr64(x, K);
    x = lazy_mul64(x, m, K);
  } else {
    for (int b = ebits - 2; b >= 0; --b) {
      x = lazy_sqr64(x, K);
      if ((e >> b) & 1) x = lazy_mul64(x, m, K);
    }
  }
  return last_mul64<PLUS>(x, kc, n, K);
}

// (m + s) mod n for m, s < n < 2^63 (no overflow of the sum).
__device__ __forceinline__ uint64_t addmod64(uint64_t m, uint64_t s, uint64_t n) {
  uint64_t t = m + s;
  return t >= n ? t - n : t;
}

// v mod n for v < 4n (n < 2^63, so 2n fits 64 bits).
__device__ __forceinline__ uint64_t mod_below_4n(uint64_t v, uint64_t n) {
  const uint64_t n2 = n << 1;
  v = v >= n2 ? v - n2 : v;
  return v >= n ? v - n : v;
}

// (w - s) mod n for w <= n, s <= n (not w = 0 with s = n).
__device__ __forceinline__ uint64_t submod64(uint64_t w, uint64_t s, uint64_t n) {
  unsigned long r;
  const bool borrow = __builtin_usubl_overflow(w, s, &r);
  return (uint64_t)r + (borrow ? n : 0ull);
}

// One skip step a s mod (2^61 - 1) for s in [1, p - 1].  The product with 8 a
// has (a s) >> 61 as its high 64 bits and 8 ((a s) mod 2^61) as its low 64
// bits, so the fold takes two shifts instead of a mask and two funnel shifts;
// 8 a < 0.75 2^64 and s < 2^61 keep the middle column below 2^64.  The sum v
// is below 2p, never 0 or p, and its bit 61 carries back in.
__device__ __forceinline__ uint64_t step_p61(uint64_t s) {
  constexpr uint64_t kA8 = 8 * kA64;
  static_assert((kA64 >> 61) == 0 && kA8 < 3ull << 62, "the middle column stays below 2^64");
  constexpr uint32_t a0 = (uint32_t)kA8, a1 = (uint32_t)(kA8 >> 32);
  const uint32_t s0 = (uint32_t)s, s1 = (uint32_t)(s >> 32);
  const uint64_t p00 = (uint64_t)s0 * a0;
  const uint64_t mid = mad_u64_u32(s1, a0, (uint64_t)s0 * a1 + (p00 >> 32));
  const uint64_t hi = (uint64_t)s1 * a1 + (mid >> 32);
  const uint64_t v = (((mid << 32) | (uint32_t)p00) >> 3) + hi;
  const uint32_t top = (uint32_t)(v >> 61);
  uint64_t r, carry;
  asm("v_mad_u64_u32 %0, %1, %2, 1, %3" : "=v"(r), "=s"(carry) : "v"(top), "v"(v & kP64));
  return r;
}

// Skip generator mod 2^61 - 1 (width 64): fold the 122-bit product.
__device__ __forceinline__ uint64_t mulmod_p61(uint64_t x, uint64_t y) {
  W128 t = mul63w(x, y);
  uint64_t lo = t.lo & kP64;
  uint64_t hi = (t.hi << 3) | (t.lo >> 61);
  uint64_t v = lo + hi;
  return v >= kP64 ? v - kP64 : v;
}

__device__ __forceinline__ uint64_t powmod_p61(uint64_t b, uint64_t e) {
  uint64_t r = 1;
  while (e) {
    if (e & 1) r = mulmod_p61(r, b);
    b = mulmod_p61(b, b);
    e >>= 1;
  }
  return r;
}

// a^t mod (2^61 - 1) computed by the whole wave: lane b contributes
// pow2[b] = a^{2^b} when bit b of t is set, and the 64 factors are multiplied
// in a butterfly (six products per lane instead of up to 61 in sequence).
// Every lane receives the result.
__device__ __forceinline__ uint64_t wave_pow_p61(const uint64_t *pow2, uint64_t t, uint32_t lane) {
  uint64_t f = (lane < 61 && ((t >> lane) & 1)) ? pow2[lane] : 1ull;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t lo = __shfl_xor((int)(uint32_t)f, d, 64);
    const uint32_t hi = __shfl_xor((int)(uint32_t)(f >> 32), d, 64);
    f = mulmod_p61(f, ((uint64_t)hi << 32) | lo);
  }
  return f;
}

// binary64(c1) / binary64(n + 1) correctly rounded, c1 = c + 1 < 2^63, with
// den = RN(n + 1), rcp = RN(1/den) and rcp_lo = RN(1/den - rcp): a rcp +
// RN(a rcp_lo) rounded once is within one ulp of a/den, and from such a
// quotient and a correctly rounded reciprocal one remainder-and-correct step
// gives the correctly rounded quotient (Markstein): four FP64 operations
// after the conversion, which rounds once (the fma).
__device__ __forceinline__ double uniform64(uint64_t c1, double den, double rcp, double rcp_lo) {
  const double a = __builtin_fma((double)(uint32_t)(c1 >> 32), 4294967296.0, (double)(uint32_t)c1);
  const double q = __builtin_fma(a, rcp, a * rcp_lo);
  return __builtin_fma(__builtin_fma(-q, den, a), rcp, q);
}

// ---- instance set-up on the device (seeding) --------------------------------

__device__ __forceinline__ uint32_t inv32(uint32_t n) {  // n^{-1} mod 2^32, n odd (Newton)
  uint32_t x = n;
  for (int i = 0; i < 5; ++i) x *= 2u - n * x;
  return x;
}

__device__ __forceinline__ uint64_t inv64(uint64_t n) {  // n^{-1} mod 2^64, n odd (Newton)
  uint64_t x = n;
  for (int i = 0; i < 6; ++i) x *= 2ull - n * x;
  return x;
}

// Montgomery power: base and result in Montgomery form, one = R mod n.
__device__ __forceinline__ uint32_t mpow32(uint32_t b, uint64_t e, uint32_t one, uint32_t n, uint32_t ninv) {
  uint32_t r = one;
  while (e) {
    if (e & 1) r = mont32(r, b, n, ninv);
    b = mont32(b, b, n, ninv);
    e >>= 1;
  }
  return r;
}

__device__ __forceinline__ uint64_t mpow64(uint64_t b, uint64_t e, uint64_t one, uint64_t n, uint64_t ninv) {
  uint64_t r = one;
  while (e) {
    if (e & 1) r = mont64(r, b, n, ninv);
    b = mont64(b, b, n, ninv);
    e >>= 1;
  }
  return r;
}

// Deterministic Rabin-Miller for odd n in [2^31, 2^32): prime bases 2..11
// decide primality below 2^32 (Sec. IV).  No base is a multiple of n.
__device__ inline bool is_prime32_dev(uint32_t n) {
  const uint32_t ninv = inv32(n);
  const uint32_t one = 0u - n;  // 2^32 mod n (n > 2^31)
  uint32_t r2 = one;            // R^2 mod n: double R mod n 32 times
  for (int i = 0; i < 32; ++i) r2 = addmod32(r2, r2, n);
  const uint32_t mone = n - one;  // Montgomery form of n - 1
  uint32_t d = n - 1;
  int s = 0;
  while ((d & 1) == 0) {
    d >>= 1;
    ++s;
  }
  const uint32_t bases[5] = {2, 3, 5, 7, 11};
  for (int i = 0; i < 5; ++i) {
    uint32_t x = mpow32(mont32(bases[i], r2, n, ninv), d, one, n, ninv);
    if (x == one || x == mone) continue;
    bool witness = true;
    for (int j = 1; j < s; ++j) {
      x = mont32(x, x, n, ninv);
      if (x == mone) {
        witness = false;
        break;
      }
    }
    if (witness) return false;
  }
  return true;
}

// Deterministic Rabin-Miller for odd n in [2^62, 2^63): the twelve prime
// bases 2..37 decide primality below 2^64 (Sec. IV).
__device__ inline bool is_prime64_dev(uint64_t n) {
  const uint64_t ninv = inv64(n);
  uint64_t one = 0ull - n;  // 2^64 - n, then reduce: 2^64 mod n
  while (one >= n) one -= n;
  uint64_t r2 = one;
  for (int i = 0; i < 64; ++i) r2 = addmod64(r2, r2, n);
  const uint64_t mone = n - one;
  uint64_t d = n - 1;
  int s = 0;
  while ((d & 1) == 0) {
    d >>= 1;
    ++s;
  }
  const uint32_t bases[12] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
  for (int i = 0; i < 12; ++i) {
    uint64_t x = mpow64(mont64(bases[i], r2, n, ninv), d, one, n, ninv);
    if (x == one || x == mone) continue;
    bool witness = true;
    for (int j = 1; j < s; ++j) {
      x = mont64(x, x, n, ninv);
      if (x == mone) {
        witness = false;
        break;
      }
    }
    if (witness) return false;
  }
  return true;
}

// j-th output (j = 0, 1, ...) of the SplitMix64 stream started at `seed`
// (Steele, Lea and Flood, 2014): the state after j+1 steps, finalised.
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t j) {
  uint64_t z = seed + (j + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// ---- wave helpers ---------------------------------------------------------

// Load of a record that no kernel writes while this one runs, at an address
// that is the same in every lane: through the constant address space, so that
// the compiler reads it with scalar loads into SGPRs and the arithmetic on it
// runs on the scalar unit instead of in every lane.
template <typename T>
__device__ __forceinline__ T const_load(const T *p) {
  static_assert(sizeof(T) % 8 == 0, "records of whole 64-bit words");
  using CP = const __attribute__((address_space(4))) uint64_t *;
  const CP q = (CP)p;
  T out;
  uint64_t *o = reinterpret_cast<uint64_t *>(&out);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 8); ++i) o[i] = q[i];
  return out;
}

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
  uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int src) {
  uint32_t lo = __shfl((int)(uint32_t)v, src, 64);
  uint32_t hi = __shfl((int)(uint32_t)(v >> 32), src, 64);
  return ((uint64_t)hi << 32) | lo;
}

// The value of lane LANE, in scalar registers.
template <int LANE>
__device__ __forceinline__ uint64_t lane_u64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, LANE);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), LANE);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int mask) {
  uint32_t lo = __shfl_xor((int)(uint32_t)v, mask, 64);
  uint32_t hi = __shfl_xor((int)(uint32_t)(v >> 32), mask, 64);
  return ((uint64_t)hi << 32) | lo;
}

// Lane value moved by a DPP control word; lanes without a source (and rows
// outside ROWS) get 0.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xf, false);
  return ((uint64_t)hi << 32) | lo;
}

// Inclusive prefix sum of v over the lanes of the wave, all lanes active:
// shifts by 1, 2, 4, 8 inside the rows of 16 lanes, then the last lane of a
// row (of two rows) added to the next ones.  Six register moves without the
// LDS round trip that a shuffle takes.
__device__ __forceinline__ uint64_t wave_inclusive_sum(uint64_t v) {
  v += dpp_u64<0x111, 0xf>(v);  // row_shr:1
  v += dpp_u64<0x112, 0xf>(v);  // row_shr:2
  v += dpp_u64<0x114, 0xf>(v);  // row_shr:4
  v += dpp_u64<0x118, 0xf>(v);  // row_shr:8
  v += dpp_u64<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_u64<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Sum of v over the 64 lanes of the wave, mod n (v < n < 2^63); every lane
// receives it.
__device__ __forceinline__ uint64_t wave_sum_mod(uint64_t v, uint64_t n) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t t = v + shfl_xor_u64(v, d);
    v = t >= n ? t - n : t;
  }
  return v;
}

// Exclusive prefix sum of v over the lanes of the wave, mod n (v < n < 2^63),
// all lanes active: the DPP steps of wave_inclusive_sum, reduced at each.
__device__ __forceinline__ uint64_t wave_exclusive_mod(uint64_t v, uint64_t n) {
  uint64_t incl = v;
  incl = addmod64(incl, dpp_u64<0x111, 0xf>(incl), n);
  incl = addmod64(incl, dpp_u64<0x112, 0xf>(incl), n);
  incl = addmod64(incl, dpp_u64<0x114, 0xf>(incl), n);
  incl = addmod64(incl, dpp_u64<0x118, 0xf>(incl), n);
  incl = addmod64(incl, dpp_u64<0x142, 0xa>(incl), n);
  incl = addmod64(incl, dpp_u64<0x143, 0xc>(incl), n);
  return submod64(incl, v, n);
}

// Orders this wave's LDS accesses across lanes (all lanes of one wave).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace dev
}  // namespace phprng
