// Gumbel keys of the random eviction (NaCl Section 5.2): a token's key is
// binary32(log-weight + g) with g = -ln(-ln u) in binary64,
// u = (word + 1/2) / 2^32 and word = Philox4x32-10 output j mod 4 at counter
// (j / 4, h, b, layer) under key = seed.  Keys are stored as order-preserving
// uint32 bits.  Shared by the stand-alone key kernel and the column
// reduction, which draws the keys of its chunk when it runs inside a whole
// eviction.
#pragma once

#include "device_common.h"
#include "philox.h"

namespace nacl {

// A binary64 constant made where it stands.  As plain constants the compiler
// keeps those of the logarithms in registers from the start of a kernel on (18
// vector and 18 scalar ones), and the score kernels, which draw keys at the end
// of their items only, spilled others for them: 32 heads of 32k keys, 128 rows
// 171 us with, 151 without; a whole eviction of 128 such heads 573 and 558.
template <uint64_t BITS>
__device__ __forceinline__ double constant_here() {
  uint32_t lo, hi;
  asm volatile("v_mov_b32 %0, %2\n\tv_mov_b32 %1, %3" : "=&v"(lo), "=v"(hi) : "n"((uint32_t)BITS), "n"((uint32_t)(BITS >> 32)));
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
#define NACL_HERE(x) constant_here<__builtin_bit_cast(uint64_t, (double)(x))>()

// ln(x) in binary64 for x >= 0 (ln 0 = -inf, ln inf = inf), to within a
// few units in the last place: x = m 2^e with m in [sqrt(1/2), sqrt(2)),
// ln m = 2 atanh(s) with s = (m - 1) / (m + 1), |s| < 0.172, summed as the
// odd series 2 s (1 + s^2/3 + s^4/5 + ... + s^20/21) (the next term is
// below 2^-59 relative), and e ln 2 added in two parts (ln 2 rounded to
// binary64 and the rest).  The quotient takes a hardware reciprocal, two
// Newton steps and one residual correction.  The keys are rounded to
// binary32 afterwards, so a few binary64 units never matter except for a
// key within that distance of a binary32 rounding boundary.
__device__ __forceinline__ double ln_f64(double x) {
  constexpr double kLn2 = 0.6931471805599453094172321;         // rounded to binary64
  constexpr double kLn2Rest = 2.319046813846299558e-17;        // ln 2 - kLn2
  constexpr double kSqrtHalf = 0.70710678118654752440;
  double m = __builtin_amdgcn_frexp_mant(x);                   // [1/2, 1)
  int e = __builtin_amdgcn_frexp_exp(x);
  if (m < kSqrtHalf) {
    m *= 2.0;
    --e;
  }
  const double f = m - 1.0;                                    // exact
  const double d = f + 2.0;
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  r = fma(r, fma(-d, r, 1.0), r);
  double s = f * r;
  s = fma(fma(-s, d, f), r, s);
  const double z = s * s;
  double q = NACL_HERE(1.0 / 21);
  q = fma(q, z, NACL_HERE(1.0 / 19));
  q = fma(q, z, NACL_HERE(1.0 / 17));
  q = fma(q, z, NACL_HERE(1.0 / 15));
  q = fma(q, z, NACL_HERE(1.0 / 13));
  q = fma(q, z, NACL_HERE(1.0 / 11));
  q = fma(q, z, NACL_HERE(1.0 / 9));
  q = fma(q, z, NACL_HERE(1.0 / 7));
  q = fma(q, z, NACL_HERE(1.0 / 5));
  q = fma(q, z, NACL_HERE(1.0 / 3));
  const double s2 = 2.0 * s;
  const double lnm = fma(s2 * z, q, s2);
  const double ed = (double)e;
  const double p = ed * kLn2;
  const double perr = fma(ed, kLn2, -p);                       // exact rounding error of p
  const double res = p + (lnm + fma(ed, kLn2Rest, perr));
  if (x == 0.0) return -INFINITY;
  if (x == INFINITY) return INFINITY;
  return res;
}

struct LnConstants {
  double ln2_hi, ln2_lo;  // 32 leading bits of ln 2, and the rest
  double q[7];            // the polynomial's coefficients, highest first
};
__device__ __forceinline__ LnConstants ln_constants() {
  return LnConstants{NACL_HERE(0.6931471803691238),   NACL_HERE(1.9082149292705877e-10),
                     {NACL_HERE(0.07308292712444311), NACL_HERE(0.07665855309105386), NACL_HERE(0.09091444727837474),
                      NACL_HERE(0.11111105565129939), NACL_HERE(0.14285714313001635), NACL_HERE(0.19999999999949722),
                      NACL_HERE(0.3333333333333335)}};
}

// ln(x) - bias ln 2 in binary64 for positive finite normal x: the logarithm of
// the uniform draw and of its exponential variate, which are all a key takes
// unless the weights are F.  ln_f64's steps with fewer instructions (the key
// kernel is bound by their issue): exponent and mantissa by integer
// arithmetic on the high word, a polynomial of degree 6 in s^2 interpolating
// (atanh(s) / s - 1) / s^2 at the Chebyshev nodes (relative error of the
// logarithm below 2^-57) where the series takes 10 terms, one Newton step (the
// residual correction squares its error again), ln 2 in two parts of which the
// first has 32 bits (exact products), and no cases for 0 and infinity.  Over
// 6e7 draws, both tails included: largest relative error 2.22e-16 (ln_f64
// 2.27e-16), mean error of a key 7.88e-17 (8.02e-17), the same binary32 keys.
// 4.2 M keys: 18.4 us before, now 14.7.
__device__ __forceinline__ double ln_pos_f64(double x, int bias, const LnConstants& c) {
  const uint64_t bits = __builtin_bit_cast(uint64_t, x);
  const uint32_t hi = (uint32_t)(bits >> 32);
  const uint32_t t = hi - 0x3FE6A09Eu;                         // mantissa into [sqrt(1/2), sqrt(2))
  const double m = __builtin_bit_cast(double, ((uint64_t)(hi - (t & 0xFFF00000u)) << 32) | (uint32_t)bits);
  const double e = (double)(((int32_t)t >> 20) - bias);
  const double f = m - 1.0, d = m + 1.0;                       // f is exact
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  double s = f * r;
  s = fma(fma(-s, d, f), r, s);
  const double z = s * s;
  double q = c.q[0];
#pragma unroll
  for (int i = 1; i < 7; ++i) q = fma(q, z, c.q[i]);
  const double s2 = s + s;
  return fma(e, c.ln2_hi, s2 + fma(s2 * z, q, e * c.ln2_lo));
}

#undef NACL_HERE

// Key of one token.  MODE selects the log-weight: 0 = F (weights
// Softmax(F)), 1 = ln F (weights F), 2 = none (uniform).
template <int MODE>
__device__ __forceinline__ uint32_t gumbel_order_key(float f, uint32_t word, const LnConstants& c) {
  // word + 1/2, from the bits of 2^52 + word.
  const double u32 = __builtin_bit_cast(double, 0x4330000000000000ull | word) - (0x1p52 - 0.5);
  const double g = -ln_pos_f64(-ln_pos_f64(u32, 32, c), 0, c);
  double key = g;
  if constexpr (MODE == 0) key = (double)f + g;
  if constexpr (MODE == 1) key = ln_f64((double)f) + g;
  return float_order_key((float)key);
}

// The keys of tokens j0 .. j0 + n - 1 (j0 a multiple of 4, n <= 4: one
// Philox block) of head (b, h) with scores f[0 .. n), into out[0 .. n).
// `mode` is uniform across the calling wave.
__device__ __forceinline__ void gumbel_block_keys(int mode, int j0, int n, int b, int h, uint32_t layer,
                                                  uint32_t k0, uint32_t k1, const float (&f)[4],
                                                  uint32_t (&out)[4]) {
  const U32x4 w = philox4x32_10(U32x4{(uint32_t)(j0 >> 2), (uint32_t)h, (uint32_t)b, layer}, k0, k1);
  const uint32_t word[4] = {w.x, w.y, w.z, w.w};
  const LnConstants c = ln_constants();
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (e < n) {
      if (mode == 0) out[e] = gumbel_order_key<0>(f[e], word[e], c);
      else if (mode == 1) out[e] = gumbel_order_key<1>(f[e], word[e], c);
      else out[e] = gumbel_order_key<2>(f[e], word[e], c);
    }
  }
}

}  // namespace nacl
