// trig.h -- fp64 sine and cosine for the hot path.
//
// sincos_fast(x): both functions of one argument.  Positions on the hot path
// stay within a few box edges of the origin, so the full-range reduction of
// the device math library (Payne-Hanek) is replaced for |x| <= 2^19 by
//   k = nearest integer to x * 2/pi,  r = x - k*pi/2  with pi/2 as the sum
//   of three doubles, one fma each.  The first is exact: pi/2's leading double
//   is a multiple of 2^-52, so is x (or k is 0 or 1 and the difference is a
//   multiple of 2^-53), and |r| < 1 leaves at most 53 bits.  The second rounds
//   once, and the third adds k 2^-109, which is below that rounding except
//   where x is next to a multiple of pi/2 and r is tiny: there it is what
//   keeps r's relative error at one ulp (two doubles alone are up to 5e4 ulp
//   off at the doubles nearest k pi/2, k < 2^18.4).  k comes from one fma that
//   adds 1.5 * 2^52, whose low word holds k.
// The sine and cosine of |r| <= pi/4 are minimax polynomials of degree 13 and
// 14 (gen_trig_constants.py; largest errors 3.4e-18 of the sine and 4.7e-20),
// evaluated by Horner's rule.  The quadrant k mod 4 picks and signs the
// results.  Arguments outside that range, infinities and NaNs go to the
// device library's sincos.
//
// sincos_shift(x, sin x, cos x, d): both functions of x + d for a small shift
// |d| <= 1/64, as the rotation by d written as three shears,
//   a = s + tan(d/2) c,  c' = c - sin(d) a,  s' = a + tan(d/2) c',
// one fma each (the product of the shears is the rotation, exactly), with
// sin d and tan(d/2) from minimax polynomials (errors below 4e-18 absolute).
// The cosine takes one rounding of its own size and the sine two, where the
// angle-addition formulas take two each, and an instruction more.  A time
// step moves a particle by dt*u, far less than 1/64 for the step sizes of
// interest, so the midpoint and end-point values of a step come from the
// start-point values without a second reduction.  Where shifts may exceed
// 1/64 longer polynomials take every shift up to 1/8, and larger shifts fall
// back to sincos_fast(x + d) (see the tiers below).  The shift uses the exact
// sum x + d, which differs from the rounded sum by at most half an ulp of x.
//
// The field integrators are bound by fp64 issue or close to it.  Against a
// quadrant by rint, Taylor series two terms longer and angle addition, with
// pi/2 in two constants: 50 fused RK2 steps of 1e7 particles 2.44 -> 2.24 ms,
// RK4 0.926 -> 0.886 ms per 10 steps of 6e6, the streaming RK2 step 1.013 ->
// 0.973 ms at 1e8, forward and adjoint of 1e7 x 200 steps 19.2 -> 18.1 ms.
// The third constant costs about 1% of that again (1.93 -> 1.96, 0.832 ->
// 0.838, 0.958 -> 0.965 and 14.53 -> 14.54 ms beside later changes).
//
// Measured on the host: within 2 ulp for |x| up to 2^19, against glibc over
// seeded arguments and against integers of 400 bits at the doubles next to the
// multiples of pi/2, and the shifted forms within one ulp of 1 in absolute
// error.
// The GPU's results equal the host build's bit for bit (both are chains of
// correctly rounded fmas).
#pragma once

#include <hip/hip_runtime.h>

namespace soax {
namespace trig {

constexpr double kPio2Hi = 0x1.921fb54442d18p+0;
constexpr double kPio2Lo = 0x1.1a62633145c07p-54;
constexpr double kPio2Tail = -0x1.f1976b7ed8fbcp-110;
constexpr double kTwoOverPi = 0x1.45f306dc9c883p-1;
constexpr double kRoundMagic = 0x1.8p52;
constexpr double kFastMax = 0x1p19;
constexpr double kShiftMax = 1.0 / 64;

// sin r = r + r^3 (S1 + w (S2 + ... + w S6)),  w = r^2
constexpr double S1 = -0x1.5555555555549p-3, S2 = 0x1.111111110f881p-7,
                 S3 = -0x1.a01a019c126d5p-13, S4 = 0x1.71de3578757cep-19,
                 S5 = -0x1.ae5e66d53a55ap-26, S6 = 0x1.5d932f420ae31p-33;
// cos r = 1 - w/2 + w^2 (C1 + w (C2 + ... + w C6))
constexpr double C1 = 0x1.555555555554cp-5, C2 = -0x1.6c16c16c15184p-10,
                 C3 = 0x1.a01a019cb26f0p-16, C4 = -0x1.27e4f80a75f0cp-22,
                 C5 = 0x1.1ee9ec4730a58p-29, C6 = -0x1.8faeced46d067p-37;

struct SinCos {
  double s, c;
};

// The two polynomials' Horner chains in w: ps = S1 + w (S2 + ... + w S6) and
// pc = C1 + w (C2 + ... + w C6), each step one fma.  On the GPU both chains
// run interleaved in one block of three-operand fmas (the top step's added
// constant from a vector register, every other constant a scalar-register
// operand): the compiler cannot see into separate asm statements and pads
// each dependent pair of them with a wait, which one block does not need.
__host__ __device__ __forceinline__ void sin_cos_series(double w, double& ps, double& pc) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("v_fma_f64 %0, %2, %3, %4\n\t"
      "v_fma_f64 %1, %2, %5, %6\n\t"
      "v_fma_f64 %0, %2, %0, %7\n\t"
      "v_fma_f64 %1, %2, %1, %8\n\t"
      "v_fma_f64 %0, %2, %0, %9\n\t"
      "v_fma_f64 %1, %2, %1, %10\n\t"
      "v_fma_f64 %0, %2, %0, %11\n\t"
      "v_fma_f64 %1, %2, %1, %12\n\t"
      "v_fma_f64 %0, %2, %0, %13\n\t"
      "v_fma_f64 %1, %2, %1, %14"
      : "=&v"(ps), "=&v"(pc)
      : "v"(w), "s"(S6), "v"(S5), "s"(C6), "v"(C5), "s"(S4), "s"(C4), "s"(S3), "s"(C3),
        "s"(S2), "s"(C2), "s"(S1), "s"(C1));
#else
  ps = fma(w, fma(w, fma(w, fma(w, fma(w, S6, S5), S4), S3), S2), S1);
  pc = fma(w, fma(w, fma(w, fma(w, fma(w, C6, C5), C4), C3), C2), C1);
#endif
}

// Out-of-range arguments: kept out of line so the fast path stays small.  The
// pair is returned by value so that the caller's results never have to live
// in memory.
inline __host__ __device__ __attribute__((noinline)) SinCos sincos_wide(double x) {
  SinCos r;
  sincos(x, &r.s, &r.c);
  return r;
}

// True where sincos_core does not hold: |x| > kFastMax, infinities, NaNs.
__host__ __device__ __forceinline__ bool beyond_fast(double x) { return !(fabs(x) <= kFastMax); }

// Both functions of |x| <= kFastMax.
__host__ __device__ __forceinline__ void sincos_core(double x, double* s, double* c) {
  const double t = fma(x, kTwoOverPi, kRoundMagic);
  const double k = t - kRoundMagic;
  const double r = fma(-k, kPio2Tail, fma(-k, kPio2Lo, fma(-k, kPio2Hi, x)));
  const double w = r * r;
  double ps, pc;
  sin_cos_series(w, ps, pc);
  const double sr = fma(r * w, ps, r);
  const double cr = fma(w, fma(w, pc, -0.5), 1.0);
  // x = k pi/2 + r:  sin x = (sr, cr, -sr, -cr)[k mod 4], cos x = (cr, -sr, -cr, sr)[k mod 4]
  const uint32_t q = static_cast<uint32_t>(__builtin_bit_cast(uint64_t, t));
  // bit 0 of q (swap sr and cr) and bit 1 (the sine's sign) moved to bit 31;
  // the cosine's sign is bit 1 of q + 1, i.e. bit 1 xor bit 0
  const uint32_t odd = q << 31;
  const uint32_t hs = (q << 30) & 0x80000000u;
  const uint32_t hc = hs ^ odd;
  const double a = odd ? cr : sr;
  const double b = odd ? sr : cr;
  *s = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, a) ^ (static_cast<uint64_t>(hs) << 32));
  *c = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, b) ^ (static_cast<uint64_t>(hc) << 32));
}

__host__ __device__ __forceinline__ void sincos_fast(double x, double* s, double* c) {
  if (beyond_fast(x)) {
    const SinCos r = sincos_wide(x);
    *s = r.s;
    *c = r.c;
    return;
  }
  sincos_core(x, s, c);
}

// |d| <= 1/64: sin d = d (1 + w (T1 + w T2)), tan(d/2) = d (1/2 + w (U1 + w U2)),  w = d^2
constexpr double T1 = -0x1.5555555528856p-3, T2 = 0x1.1110803b544a5p-7;
constexpr double U1 = 0x1.55555553d8698p-5, U2 = 0x1.111378a2960cfp-8;
// |d| <= 1/8: the same with four terms each
constexpr double kShiftLong = 1.0 / 8;
constexpr double V1 = -0x1.5555555555552p-3, V2 = 0x1.1111111107f30p-7,
                 V3 = -0x1.a019ffe78712fp-13, V4 = 0x1.71bd73cf1a7dbp-19;
constexpr double W1 = 0x1.5555555554b28p-5, W2 = 0x1.1111111d6c97dp-8,
                 W3 = 0x1.ba1b0c8520afdp-12, W4 = 0x1.67b2237a761e5p-15;

// What the caller guarantees about the shift, by tier.  kTierSmall:
// |d| <= kShiftMax; the short polynomials.  kTierMid: |d| <= kShiftLong; the
// longer ones for every shift (no branch, so the lanes of a wave never
// split between two forms).  kTierAny: any d; the longer polynomials up to
// kShiftLong and a full reduction of x + d beyond it.  Where its guarantee
// holds, kTierMid gives exactly the results of kTierAny.
constexpr int kTierSmall = 0;
constexpr int kTierMid = 1;
constexpr int kTierAny = 2;

template <int TIER = kTierAny>
__host__ __device__ __forceinline__ void sincos_shift(double x, double sx, double cx, double d,
                                                      double* s, double* c) {
  double p, q;  // sin d / d and tan(d/2) / d
  const double w = d * d;
  if (TIER == kTierSmall) {
    p = fma(w, fma(w, T2, T1), 1.0);
    q = fma(w, fma(w, U2, U1), 0.5);
  } else {
    if (TIER == kTierAny && !(fabs(d) <= kShiftLong)) {
      sincos_fast(x + d, s, c);
      return;
    }
    p = fma(w, fma(w, fma(w, fma(w, V4, V3), V2), V1), 1.0);
    q = fma(w, fma(w, fma(w, fma(w, W4, W3), W2), W1), 0.5);
  }
  const double sd = d * p, th = d * q;
  const double a = fma(th, cx, sx);
  const double c1 = fma(-sd, a, cx);
  *s = fma(th, c1, a);
  *c = c1;
}

}  // namespace trig
}  // namespace soax
