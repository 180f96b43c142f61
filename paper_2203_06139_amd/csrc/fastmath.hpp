// fastmath.hpp -- lean FP64 elementary functions for the per-bin sweep.
//
// On gfx950 FP64 FMA issues at the full (non-packed) vector rate, so the cost
// of a bin is its VALU instruction count.  The library versions of exp, log
// and division carry range/special-case handling that the objective never
// needs (its arguments are finite and, where it matters, positive normal), so
// these replacements drop it:
//   exp_fast   Cody-Waite reduction by ln 2 and a degree-13 Taylor polynomial
//              on |r| <= ln2/2 (truncation < 1e-17); inputs below -746 give 0.
//   rcp_fast   v_rcp_f64 seed (measured on gfx950: <= 4.7e-8 relative) and
//              one Newton step (<= 2.3e-15); div_fast adds one residual
//              correction, which brings the quotient to about 1 ulp (the
//              refinement the compiler's IEEE division uses, without its
//              scaling for extreme exponents).
//   exp_hw32   the FP32 hardware exp2, for the FP32-per-bin variant: results
//              below about e^-87 are 0 and above e^88 infinite.
//   log_lut    x = 2^e m, m in [0.75, 1.5), so that arguments just below 1 do
//              not cancel against ln 2; a 1024-entry LDS table of 1/c and ln c
//              at the midpoints c of the top 10 mantissa bits gives f = m/c - 1
//              with |f| < 2^-11, and ln(1+f) is a degree-4 polynomial
//              (|f|^5/5 < 1e-17).  log_lut(0) is finite (about -709): an
//              empty bin's n ln(n/mu) term is 0 * finite = 0.
//   erf_from_phi  erf where exp(-z^2/2) is needed beside it.
// Inputs must be finite; div_fast needs a positive normal divisor.
#pragma once

#include <hip/hip_runtime.h>

namespace hf {

constexpr double kLog2e = 1.4426950408889634074;
// ln 2 split so that k * kLn2Hi is exact for |k| < 2^11 (trailing zero bits).
constexpr double kLn2Hi = 6.93147180369123816490e-01;
constexpr double kLn2Lo = 1.90821492927058770002e-10;
constexpr double kLn2 = 6.93147180559945309417e-01;

constexpr int kLogLutBits = 10;
constexpr int kLogLut = 1 << kLogLutBits;

__device__ __forceinline__ double exp_fast(double x) {
  x = fmax(x, -746.0);
  const double k = __builtin_rint(x * kLog2e);
  double r = fma(-k, kLn2Hi, x);
  r = fma(-k, kLn2Lo, r);
  double p = 1.0 / 6227020800.0;     // 1/13!
  p = fma(p, r, 1.0 / 479001600.0);  // 1/12!
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return __builtin_amdgcn_ldexp(p, static_cast<int>(k));
}

// 2^(-u^2) of N values in step: a Gaussian whose width has the factor
// sqrt(2 ln 2) taken in (kGaussU), so that nothing is left to scale.  -u^2 is
// split without rounding into the nearest integer (read from the low word of
// the sum with 1.5 2^52) and r in [-0.5, 0.5], where 2^r is a polynomial of
// degree 11 (the Chebyshev interpolant of (2^r - 1)/r, computed in 60-digit
// arithmetic; error 2e-17): 16 operations against exp_fast's 22 with its
// argument.  A chain of dependent FP64 operations issues one in about nine
// slots, so the chains of several values run side by side; the compiler keeps
// the order that it is given.
constexpr double kGaussU = 8.49321800288019068681e-01;     // sqrt(log2(e) / 2)
constexpr double kGaussULo = -2.59594641045974034667e-17;  // and its remainder
constexpr double kGaussUInv2 = 1.38629436111989057245e+00;    // kGaussU^-2
constexpr double kGaussUInv2Lo = 4.63809362769259911684e-17;
constexpr double kGaussUInv3 = 1.63223687493924596303e+00;    // kGaussU^-3
constexpr double kGaussUInv3Lo = 5.25745411534361271364e-17;

// kGaussU / s to the last bit, from is = 1 / s.
__device__ __forceinline__ double gauss_unit(double is, double s) {
  const double q = kGaussU * is;
  return fma(is, fma(-q, s, kGaussU) + kGaussULo, q);
}

template <int N>
__device__ __forceinline__ void gauss_n(const double (&u)[N], double (&e)[N]) {
  constexpr double kRound = 6755399441055744.0;
  constexpr double c[] = {7.07258594926922338728e-09, 1.01780624458457736676e-07,
                          1.32154425879216893033e-06, 1.52527338298361192352e-05,
                          1.54035304417360498870e-04, 1.33335581464169355623e-03,
                          9.61812910760688824507e-03, 5.55041086648215969968e-02,
                          2.40226506959100971628e-01, 6.93147180559945286227e-01,
                          1.0};
  double r[N], p[N];
  int n[N];
#pragma unroll
  for (int i = 0; i < N; ++i) r[i] = fmin(fabs(u[i]), 44.0);  // 2^(-44^2) is 0
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double k = fma(-r[i], r[i], kRound);
    n[i] = __double2loint(k);
    r[i] = fma(-r[i], r[i], kRound - k);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) p[i] = fma(4.45496059818651856354e-10, r[i], c[0]);
#pragma unroll
  for (int j = 1; j < 11; ++j)
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = fma(p[i], r[i], c[j]);
#pragma unroll
  for (int i = 0; i < N; ++i) e[i] = __builtin_amdgcn_ldexp(p[i], n[i]);
}

// e^x - 1 with the same reduction, x = k ln 2 + r: 2^k (e^r - 1) + (2^k - 1),
// accurate relative to itself down to x = 0.
__device__ __forceinline__ double expm1_fast(double x) {
  x = fmax(x, -746.0);
  const double k = __builtin_rint(x * kLog2e);
  double r = fma(-k, kLn2Hi, x);
  r = fma(-k, kLn2Lo, r);
  double p = 1.0 / 6227020800.0;     // 1/13!
  p = fma(p, r, 1.0 / 479001600.0);  // 1/12!
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r * r, r);
  const double s = __builtin_amdgcn_ldexp(1.0, static_cast<int>(k));
  return fma(s, p, s - 1.0);
}

// e^x through the FP32 hardware exp2 (about 1e-7 relative for |x| < 8).
__device__ __forceinline__ double exp_hw32(double x) {
  return static_cast<double>(__builtin_amdgcn_exp2f(static_cast<float>(x * kLog2e)));
}

__device__ __forceinline__ double rcp_fast(double d) {
  const double y = __builtin_amdgcn_rcp(d);
  return fma(y, fma(-d, y, 1.0), y);
}

// a / d for a positive normal d.  The FP32-per-bin variant keeps the FP64
// seed (an FP32 seed would overflow or vanish for divisors outside FP32's
// range) and drops the residual correction (2.3e-15 relative is ample there).
template <bool F32BIN>
__device__ __forceinline__ double div_fast(double a, double d) {
  const double y = rcp_fast(d);
  const double q = a * y;
  return F32BIN ? q : fma(fma(-d, q, a), y, q);
}

// Clamp of a recurrence ratio's exponent: 0 * exp(a) must stay 0, so exp(a)
// must stay finite in the precision it is taken in (e^88.7 overflows FP32).
template <bool F32BIN>
__device__ __forceinline__ double clamp_ratio_exponent(double a) {
  constexpr double lim = F32BIN ? 80.0 : 700.0;
  return fmin(fmax(a, -lim), lim);
}

// Log table entry j: 1/c_j and ln of c_j (of c_j/2 from 1.5 up), with
// c_j = 1 + (j + 1/2)/kLogLut.  Computed once per context on the host
// (log_lut_host) and copied into each block's LDS by log_lut_load; the block
// must synchronise before the first log_lut call.
__host__ __device__ inline void log_lut_entry(int i, double* ic, double* lnc) {
  const int j = i ^ (kLogLut / 2 - 1);  // top mantissa bits of the arguments with entry i
  const double c = 1.0 + (j + 0.5) / kLogLut;
  *ic = j >= kLogLut / 2 ? 2.0 * (1.0 / c) : 1.0 / c;
  *lnc = -log(*ic);
}

__device__ __forceinline__ void log_lut_load(double2* lut, const double2* __restrict__ src) {
  for (int j = threadIdx.x; j < kLogLut; j += blockDim.x) lut[j] = src[j];
}

// Degree of the ln(1+f) polynomial: 4 terms for FP64 accuracy, 3 for the
// FP32-per-bin variant (|f|^4/4 < 1e-14).
template <bool F32BIN>
__device__ __forceinline__ double log_lut(double x, const double2* __restrict__ lut) {
  // x = 2^e m with m in [0.75, 1.5): the high word's distance below that of
  // 1.5 (in halves, where the difference cannot overflow) holds -e on top of
  // the table's index.  A negative x, of a bin with a count below zero, gets
  // ln|x| less 2048 ln 2: a constant per bin.  Six integer operations; with m
  // in [1, 2) and e corrected for the upper half of the table eight, and 4096
  // fits of uneven sizes 946 us instead of 906 with the same bits in every
  // result
  const int hi = __double2hiint(x);
  const int d = 0x1ffbffff - (hi >> 1);
  const int ne = d >> 19;
  const double m = __hiloint2double(hi + (ne << 20), __double2loint(x));
  const double2 t = lut[(d >> (19 - kLogLutBits)) & (kLogLut - 1)];
  const double f = fma(m, t.x, -1.0);
  double p;
  if (F32BIN) {
    p = 1.0 / 3.0;
    p = fma(p, f, -0.5);
    p = fma(p, f, 1.0);
  } else {
    p = -0.25;
    p = fma(p, f, 1.0 / 3.0);
    p = fma(p, f, -0.5);
    p = fma(p, f, 1.0);
  }
  // e ln 2 in one rounding: e = 0 for arguments in [0.75, 1.5), where the
  // objective cancels and needs the log to the last bit; elsewhere |ln x| >
  // 0.28 and the term it enters is large, so ~1e-16 relative is ample.
  const double ned = static_cast<double>(ne);
  return fma(p, f, fma(ned, -kLn2, t.y));
}

// erf(z / sqrt 2) where phi = exp(-z^2 / 2) is at hand (within a few ulp).
// With x = |z| / sqrt 2: below 1, x times a polynomial of degree 12 in x^2;
// from 1 on, 1 - phi erfcx(x), erfcx(x) = exp(x^2) erfc(x) as t times a
// polynomial of degree 15 in t = 1/(x + 3), mapped to u in [-1, 1] over x =
// 1..6 (in the manner of Shepherd & Laframboise, Math. Comp. 36, 1981, who
// expand erfcx in (x - k)/(x + k)); beyond 6 the result is 1.  Both are
// Chebyshev interpolants computed in 60-digit arithmetic (truncation below
// 1e-17).  Absolute error, against 50 digits: rms 3.5e-17, at most 1.1e-16, as
// of the library's erf, which takes about 200 instructions to these 20 to 35.
constexpr int kErfNear = 13, kErfFar = 16;  // coefficients, highest first
static __device__ const double kErfCoef[kErfNear + kErfFar] = {
    5.957176147748911e-11, -1.1372848856791674e-09, 1.4659775274047436e-08,
    -1.6350312701054695e-07, 1.6461000484121368e-06, -1.4925595266831182e-05,
    0.0001205533111164271, -0.000854832698083379, 0.0052239776248180145, -0.026866170645076792,
    0.11283791670954879, -0.3761263890318375, 1.1283791670955126,
    -2.279742613773115e-12, 5.830884699677111e-12, 8.098927716409088e-11, -2.9728506949500295e-10,
    -2.942735833696472e-09, 1.1449481840693569e-08, 1.3353032032709014e-07,
    -2.8199389473825003e-07, -7.246255012285937e-06, -1.608776475267465e-05,
    0.00032354378790109227, 0.003933868783798848, 0.025474072799978032, 0.11683673753802074,
    0.4118820962100305, 1.1519074596928367,
};

// c: kErfCoef in LDS.  As literals the coefficients outlive the scalar
// registers and are held in 58 vector registers through the whole kernel.
__device__ __forceinline__ double erf_from_phi(double z, double phi, const double* c) {
  const double x = fabs(z) * 0.70710678118654752440;
  double r;
  // neighbouring bins mostly fall on one side, so a wave takes one branch;
  // with both forms evaluated and selected 1e6 bins took 23.0 us, not 19.5
  if (x < 1.0) {
    const double w = x * x;
    double p = c[0];
#pragma unroll
    for (int k = 1; k < kErfNear; ++k) p = fma(p, w, c[k]);
    r = p * x;
  } else {
    const double xc = x > 6.0 ? 6.0 : x;  // keeps a NaN
    const double d = xc + 3.0;
    double t = rcp_fast(d);
    t = fma(t, fma(-d, t, 1.0), t);
    const double u = fma(t, 14.4, -2.6);
    double q = c[kErfNear];
#pragma unroll
    for (int k = 1; k < kErfFar; ++k) q = fma(q, u, c[kErfNear + k]);
    r = fma(-q * t, phi, 1.0);
  }
  return __builtin_copysign(r, z);
}

// To LDS; the block must synchronise before the first use.
__device__ __forceinline__ void erf_load(double* c) {
  if (threadIdx.x < kErfNear + kErfFar) c[threadIdx.x] = kErfCoef[threadIdx.x];
}

// S(u) = sinh(u)/u and S'(u) = (cosh u - S(u))/u: the average of
// exp(b0 + b1 t) over [t_c - d, t_c + d] is exp(b0 + b1 t_c) S(b1 d).  Taylor
// series to u^10 for |u| < 1/2 (truncation below 4e-14 relative), the
// closed forms beyond, where cosh u - S(u) no longer cancels badly.
__device__ __forceinline__ void sinhc(double u, double& S, double& dS) {
  if (fabs(u) < 0.5) {
    const double u2 = u * u;
    S = 1.0 + u2 / 6.0 * (1.0 + u2 / 20.0 * (1.0 + u2 / 42.0 * (1.0 + u2 / 72.0 * (1.0 + u2 / 110.0))));
    dS = u / 3.0 * (1.0 + u2 / 10.0 * (1.0 + u2 / 28.0 * (1.0 + u2 / 54.0 * (1.0 + u2 / 88.0))));
  } else {
    S = sinh(u) / u;
    dS = (cosh(u) - S) / u;
  }
}

}  // namespace hf
