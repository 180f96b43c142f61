// unbinned.hpp -- extended unbinned NLL and its reverse-mode gradient:
// the binned objective's per-bin code applied to single events at arbitrary
// positions (the per-event batch evaluation of RooFit-style likelihoods).
//
// For events x_e with weights w_e (default 1) and the 1D Gauss + polynomial
// or exponential model read as an intensity lambda(x; theta):
//   L(theta) = Lambda(theta) - sum_e w_e ln lambda(x_e),
//   Lambda   = integral of lambda over [lo, hi]   (the expected count),
// the extended likelihood of a Poisson process (the binned Poisson objective
// as the bins shrink to single events).  Per event the forward sweep
// evaluates lambda, the reverse sweep with adjoint -w/lambda accumulates
// dlambda/dtheta (without the 1/s of the Gaussian mean and width columns,
// applied to the totals); one exponential per Gaussian and a Newton reciprocal
// per event, and a log per event only where there are weights.  Lambda and its gradient are closed forms (per
// Gaussian with z_b = (b - m)/s, e_b = exp(-z_b^2/2)):
//   Lambda_g = A s sqrt(pi/2) [erf(z_hi/sqrt 2) - erf(z_lo/sqrt 2)],
//   d/dA = Lambda_g/A,  d/dm = A (e_lo - e_hi),
//   d/ds = Lambda_g/s + A (z_lo e_lo - z_hi e_hi);
//   polynomial: d/dc_j = t_scale (t_hi^(j+1) - t_lo^(j+1))/(j+1);
//   exponential: (hi - lo) E_c S(b1 d), E_c = exp(b0 + b1 t_c), S = sinh(u)/u;
// thread 0 of block 0 computes them into LDS during the prologue and adds
// them to the partials it publishes.  Events outside
// [lo, hi] are skipped; lambda <= 0 at an event inside is a domain error.
#pragma once

#include <type_traits>

#include "device.hpp"

namespace hf {

struct UnbinnedArgs {
  const double* x;   // [n] event positions
  const float* w;    // [n] or null
  int64_t n;
  double lo, hi;
  const double* theta;
  double* nll_out;
  double* grad_out;  // [P] or null (value only)
  int32_t* status_out;
  int32_t P;
  double t_shift, t_scale;
  double* part;
  int32_t* part_flags;
  const double2* log_lut;
};

// Launches the main kernel and returns the grid it used through *grid_used
// (the caller then launches the finishing kernel over that many partials,
// unless one block has written the outputs itself).
using UnbinnedFn = hipError_t (*)(const UnbinnedArgs&, bool vec, int num_cu, int max_grid,
                                  hipStream_t, int* grid_used);

// Event pairs per thread per step (16-byte loads of two positions); the next
// step's positions are requested while the current step is computed.  The
// kernel is bound by the issue of FP64 instructions: about 67 per event of
// two Gaussians + cubic, which take 30 us of 1e7 events where a kernel of
// nothing but as many FMAs takes 29 (reading alone takes 12.5).
// 1e7 events in us on the GPU: one event after the other, each with its own
// log and reciprocal, 49.3; the logs' product 43.1; exponentials of 4 events
// side by side 41.4; 2^(-u^2) 39.2; contiguous ranges 37.9; 2 events side by
// side and 3 waves per SIMD 36.5, with 2 pairs per step 36.4 (3 pairs 37.8,
// 4 waves with 8 spills 38.1), where 1000 events take 5.8 against 6.5.
constexpr int kUbPairs = 2;
// Events whose exponentials run side by side, and the waves per SIMD that the
// registers are to leave room for: four Gaussians would spill 4 to 28 of them
// at three waves.
template <int NG, int BKG>
constexpr int kUbSide = NG + (BKG == BKG_EXP) <= 1 ? 4 : 2;
template <int NG>
constexpr int kUbWaves = NG <= 3 ? 3 : 2;

template <bool WEIGHTED, int U>
__device__ __forceinline__ void load_pairs(const UnbinnedArgs& a, int64_t q0, int64_t end,
                                           double2 (&xv)[U], float2 (&wv)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t q = q0 + u * kBlock;
    xv[u] = make_double2(__builtin_nan(""), __builtin_nan(""));  // skipped
    wv[u] = make_float2(0.0f, 0.0f);
    if (q < end) {
      xv[u] = reinterpret_cast<const double2*>(a.x)[q];
      if constexpr (WEIGHTED) wv[u] = reinterpret_cast<const float2*>(a.w)[q];
    }
  }
}

// The product of a thread's intensities as mantissa and exponent: L needs the
// sum of their logs, which is the log of the product.  A factor costs four
// instructions (its mantissa and exponent, a product and a sum) instead of a
// log's twenty, and the log is taken once per thread.  The mantissa is brought
// back into [0.5, 1) once per step, so it stays far from underflow.
struct LogProduct {
  double m = 1.0;
  int64_t e = 0;
  __device__ __forceinline__ void times(double x, int& step_e) {
    m *= __builtin_amdgcn_frexp_mant(x);
    step_e += __builtin_amdgcn_frexp_exp(x);
  }
  __device__ __forceinline__ void end_step(int step_e) {
    e += step_e + __builtin_amdgcn_frexp_exp(m);
    m = __builtin_amdgcn_frexp_mant(m);
  }
  // ln of the product
  __device__ __forceinline__ double log(const double2* __restrict__ lut) const {
    return fma(static_cast<double>(e), kLn2, log_lut<false>(m, lut));
  }
};

// N events.  ALL: they are known to lie in the range.  WEIGHTED: the weights
// apply (else 1) and the logs are taken here; otherwise the intensities go
// into `prod`.
// us: kGaussU over each width; the Gaussians' sums are of e, e u and e u^2.
template <int NG, int BKG, bool GRAD, bool ALL, bool WEIGHTED, int N, int NV>
__device__ __forceinline__ void event_terms(const UnbinnedArgs& a, const Model1D<NG, BKG>& M,
                                            const double* us, const double2* __restrict__ lut,
                                            const double* xs, const float* ws, double (&acc)[NV],
                                            LogProduct& prod, int& step_e, int& flags) {
  using S = Shape1D<NG, BKG>;
  bool in[N];
  double x[N], t[N], lam[N];
  double u[NG > 0 ? NG * N : 1], e[NG > 0 ? NG * N : 1], eb[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    in[i] = ALL || (xs[i] >= a.lo && xs[i] <= a.hi);
    // a skipped event (outside the range, or NaN) is evaluated at the range's
    // midpoint with weight 0, where every partial is finite: at its own x a
    // polynomial power could overflow and 0 * inf would reach the sums
    x[i] = in[i] ? xs[i] : 0.5 * (a.lo + a.hi);
    t[i] = (x[i] - M.tshift) * M.ta;
#pragma unroll
    for (int g = 0; g < NG; ++g) u[NG * i + g] = (x[i] - M.m[g]) * us[g];
  }
  if constexpr (NG > 0) gauss_n(u, e);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if constexpr (BKG == BKG_EXP)
      lam[i] = eb[i] = exp_fast(fma(M.c[1], t[i], M.c[0]));
    else
      lam[i] = S::NB > 0 ? M.c[S::NB > 0 ? S::NB - 1 : 0] : 0.0;
  }
  if constexpr (BKG != BKG_EXP) {
#pragma unroll
    for (int j = S::NB - 2; j >= 0; --j)
#pragma unroll
      for (int i = 0; i < N; ++i) lam[i] = fma(lam[i], t[i], M.c[j]);
  }
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int i = 0; i < N; ++i) lam[i] = fma(M.A[g], e[NG * i + g], lam[i]);
  double r[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    // a domain error makes L infinite and the gradient NaN whatever was
    // summed, so it is only flagged; a skipped event must leave no trace
    const bool ok = lam[i] > 0.0;
    flags |= (in[i] && !ok) ? ST_DOMAIN : 0;
    const double lk = ALL ? lam[i] : (in[i] && ok ? lam[i] : 1.0);
    r[i] = rcp_fast(lk);
    if constexpr (WEIGHTED) {
      const double we = in[i] ? static_cast<double>(ws[i]) : 0.0;
      acc[0] = fma(we, log_lut<false>(lk, lut), acc[0]);
      r[i] *= we;
    } else {
      prod.times(lk, step_e);
      if constexpr (!ALL) r[i] = in[i] ? r[i] : 0.0;
    }
  }
  if constexpr (GRAD) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        // the amplitude and the width are applied to the totals
        const double re = r[i] * e[NG * i + g];
        const double ru = re * u[NG * i + g];
        acc[1 + 3 * g] += re;
        acc[2 + 3 * g] += ru;
        acc[3 + 3 * g] = fma(ru, u[NG * i + g], acc[3 + 3 * g]);
      }
      if constexpr (BKG == BKG_EXP) {
        const double rb = r[i] * eb[i];
        acc[1 + 3 * NG] += rb;
        acc[2 + 3 * NG] = fma(rb, t[i], acc[2 + 3 * NG]);
      } else {
        double rt = r[i];
#pragma unroll
        for (int j = 0; j < S::NB; ++j) {
          acc[1 + 3 * NG + j] += rt;
          if (j + 1 < S::NB) rt *= t[i];
        }
      }
    }
  }
}

// Lambda (out[0]) and dLambda/dtheta_k (out[1 + k], final values).
template <int NG, int BKG>
__device__ void lambda_terms(const UnbinnedArgs& a, const Model1D<NG, BKG>& M, double* out) {
  using S = Shape1D<NG, BKG>;
  constexpr double kRt = 1.2533141373155002512;  // sqrt(pi/2)
  constexpr double kIr2 = 0.70710678118654752440;
  double lam = 0.0;
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const double s = 1.0 / M.is[g];
    const double zl = (a.lo - M.m[g]) * M.is[g], zh = (a.hi - M.m[g]) * M.is[g];
    const double el = exp(-0.5 * zl * zl), eh = exp(-0.5 * zh * zh);
    const double ia = s * kRt * (erf(zh * kIr2) - erf(zl * kIr2));
    const double lg = M.A[g] * ia;
    lam += lg;
    out[1 + 3 * g] = ia;
    out[2 + 3 * g] = M.A[g] * (el - eh);
    out[3 + 3 * g] = lg * M.is[g] + M.A[g] * (zl * el - zh * eh);
  }
  if constexpr (BKG == BKG_EXP) {
    // (hi - lo) E_c S(b1 d) over the range, E_c at its midpoint t_c, d its
    // half-width in t (S = sinh(u)/u, see sinhc)
    const double tl = (a.lo - M.tshift) * M.ta, th = (a.hi - M.tshift) * M.ta;
    const double tc = 0.5 * (tl + th), d = 0.5 * (th - tl), w = a.hi - a.lo;
    const double Ec = exp(fma(M.c[1], tc, M.c[0]));
    double Sh, dSh;
    sinhc(M.c[1] * d, Sh, dSh);
    lam = fma(w * Ec, Sh, lam);
    out[1 + 3 * NG] = w * Ec * Sh;
    out[2 + 3 * NG] = w * Ec * fma(tc, Sh, d * dSh);
  } else if constexpr (S::NB > 0) {
    const double tl = (a.lo - M.tshift) * M.ta, th = (a.hi - M.tshift) * M.ta;
    double pl = tl, ph = th;
#pragma unroll
    for (int j = 0; j < S::NB; ++j) {
      const double ij = a.t_scale * (ph - pl) / static_cast<double>(j + 1);
      lam = fma(M.c[j], ij, lam);
      out[1 + 3 * NG + j] = ij;
      pl *= tl;
      ph *= th;
    }
  }
  out[0] = lam;
}

template <int NG, int BKG, bool GRAD, bool VEC>
__global__ __launch_bounds__(kBlock, kUbWaves<NG>) void k_nll_unbinned(UnbinnedArgs a) {
  using S = Shape1D<NG, BKG>;
  constexpr int NV = GRAD ? S::P + 1 : 1;
  __shared__ double2 lut[kLogLut];
  __shared__ double lamd[S::P + 1];
  log_lut_load(lut, a.log_lut);
  Model1D<NG, BKG> M;
  M.init(a.theta, a.t_shift, a.t_scale);
  const bool finite = all_finite(a.theta, S::P);
  if (threadIdx.x == 0 && blockIdx.x == 0) lambda_terms<NG, BKG>(a, M, lamd);
  __syncthreads();
  double us[NG > 0 ? NG : 1];
#pragma unroll
  for (int g = 0; g < NG; ++g) us[g] = gauss_unit(M.is[g], a.theta[3 * g + 2]);
  double acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  int flags = 0;
  const int64_t tid = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  LogProduct prod;
  auto events = [&](auto weighted) {
    constexpr bool W = decltype(weighted)::value;
    if constexpr (VEC) {
      // a block's pairs are contiguous and whole steps, so that only the last
      // block has lanes without events
      constexpr int64_t step = kUbPairs * kBlock;
      const int64_t steps = (a.n / 2 + step - 1) / step;
      const int64_t end = min(a.n / 2, steps * (blockIdx.x + 1) / gridDim.x * step);
      double2 xn[kUbPairs];
      float2 wn[kUbPairs];
      int64_t q0 = steps * blockIdx.x / gridDim.x * step + threadIdx.x;
      load_pairs<W>(a, q0, end, xn, wn);
      for (; q0 < end; q0 += step) {
        double xv[2 * kUbPairs];
        float wv[2 * kUbPairs];
        bool all = true;
#pragma unroll
        for (int u = 0; u < kUbPairs; ++u) {
          xv[2 * u] = xn[u].x;
          xv[2 * u + 1] = xn[u].y;
          wv[2 * u] = wn[u].x;
          wv[2 * u + 1] = wn[u].y;
          all = all && xn[u].x >= a.lo && xn[u].x <= a.hi && xn[u].y >= a.lo && xn[u].y <= a.hi;
        }
        if (q0 + step < end) load_pairs<W>(a, q0 + step, end, xn, wn);
        int step_e = 0;
        auto step_terms = [&](auto inside) {
          constexpr bool ALL = decltype(inside)::value;
          constexpr int N = kUbSide<NG, BKG>;
#pragma unroll
          for (int u = 0; u < 2 * kUbPairs; u += N)
            event_terms<NG, BKG, GRAD, ALL, W, N>(a, M, us, lut, xv + u, wv + u, acc, prod, step_e,
                                                  flags);
        };
        // the wave's events all in the range: the usual case, without selects
        if (__all(all))
          step_terms(std::true_type{});
        else
          step_terms(std::false_type{});
        prod.end_step(step_e);
      }
      if ((a.n & 1) && tid == 0) {
        int step_e = 0;
        const double x = a.x[a.n - 1];
        const float w = W ? a.w[a.n - 1] : 1.0f;
        event_terms<NG, BKG, GRAD, false, W, 1>(a, M, us, lut, &x, &w, acc, prod, step_e, flags);
        prod.end_step(step_e);
      }
    } else {
      for (int64_t e = tid; e < a.n; e += stride) {
        int step_e = 0;
        const double x = a.x[e];
        const float w = W ? a.w[e] : 1.0f;
        event_terms<NG, BKG, GRAD, false, W, 1>(a, M, us, lut, &x, &w, acc, prod, step_e, flags);
        prod.end_step(step_e);
      }
    }
    if constexpr (!W) acc[0] += prod.log(lut);
  };
  if (a.w)
    events(std::true_type{});
  else
    events(std::false_type{});
  // L = Lambda - sum w ln lambda: every block publishes -(its sums) times
  // the final factors, and block 0 adds Lambda and its derivatives
  __shared__ double fac[NV];
  if (threadIdx.x < NV) fac[threadIdx.x] = -gauss_factor(M, us, threadIdx.x);
  grid_publish<NV>(acc, flags | (finite ? 0 : ST_NONFINITE), fac, lamd, a.part, a.part_flags,
                   [&](int k, double x, int f) {
                     write_output({a.nll_out, a.grad_out, a.status_out, 0u}, k, x, f, 1.0);
                   });
}

// Blocks per CU that fit (queried once per variant) bound a single round.
template <int NG, int BKG, bool GRAD, bool VEC>
hipError_t launch_unbinned_v(const UnbinnedArgs& a, int num_cu, int max_grid, hipStream_t s,
                             int* grid_used) {
  static const int occ = [] {
    int o = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, k_nll_unbinned<NG, BKG, GRAD, VEC>, kBlock,
                                                     0) != hipSuccess || o < 1)
      o = 1;
    return o;
  }();
  const int64_t per = VEC ? 2 * kUbPairs : 1;
  const int64_t need = (a.n + per * kBlock - 1) / (per * kBlock);
  int64_t grid = static_cast<int64_t>(num_cu) * occ;
  if (grid > need) grid = need;
  if (grid > max_grid) grid = max_grid;
  if (grid < 1) grid = 1;
  *grid_used = static_cast<int>(grid);
  hipLaunchKernelGGL((k_nll_unbinned<NG, BKG, GRAD, VEC>), dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

template <int NG, int BKG>
hipError_t launch_unbinned(const UnbinnedArgs& a, bool vec, int num_cu, int max_grid,
                           hipStream_t s, int* grid_used) {
  if (a.grad_out)
    return vec ? launch_unbinned_v<NG, BKG, true, true>(a, num_cu, max_grid, s, grid_used)
               : launch_unbinned_v<NG, BKG, true, false>(a, num_cu, max_grid, s, grid_used);
  return vec ? launch_unbinned_v<NG, BKG, false, true>(a, num_cu, max_grid, s, grid_used)
             : launch_unbinned_v<NG, BKG, false, false>(a, num_cu, max_grid, s, grid_used);
}

// bkg: the background code (polynomial degree -1..3, or BKG_EXP).
template <int NG>
UnbinnedFn pick_unbinned_ng(int bkg) {
  switch (bkg) {
    case -1:
      if constexpr (NG == 0) return nullptr;
      else return &launch_unbinned<NG, BKG_NONE>;
    case 0:
      return &launch_unbinned<NG, 0>;
    case 1:
      return &launch_unbinned<NG, 1>;
    case 2:
      return &launch_unbinned<NG, 2>;
    case 3:
      return &launch_unbinned<NG, 3>;
    case BKG_EXP:
      return &launch_unbinned<NG, BKG_EXP>;
    default:
      return nullptr;
  }
}

// Defined in unbinned_ng{0..4}.hip.
UnbinnedFn pick_unbinned_ng0(int bkg);
UnbinnedFn pick_unbinned_ng1(int bkg);
UnbinnedFn pick_unbinned_ng2(int bkg);
UnbinnedFn pick_unbinned_ng3(int bkg);
UnbinnedFn pick_unbinned_ng4(int bkg);

}  // namespace hf
