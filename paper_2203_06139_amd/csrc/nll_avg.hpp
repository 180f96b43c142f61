// nll_avg.hpp -- objective (+ gradient) kernels of the bin-average 1D model
// and of histograms with bins of any widths.
//
// Bin average: mu_i is the Gauss + polynomial model's integral over bin i
// divided by the bin width, instead of its value at the bin centre (the
// "integral of the function in the bin" form of a binned fit).  Bins of any
// widths (a.x_edges: nx + 1 ascending edges): the bin-average kernel takes
// its edges from the array, and k_nll_1d_edges evaluates the centre model
// at each bin's midpoint (one exp per Gaussian and bin: the uniform grid's
// recurrences do not apply).
//
// Per Gaussian, with edges a < b of the bin, z_x = (x - m)/s and
// e_x = exp(-z_x^2/2):
//   mu_g   = A s sqrt(pi/2) [erf(z_b/sqrt 2) - erf(z_a/sqrt 2)] / h
//   dmu/dA = s sqrt(pi/2) [erf difference] / h
//   dmu/dm = A (e_a - e_b) / h
//   dmu/ds = mu_g / s + A (z_a e_a - z_b e_b) / h
// and for the polynomial in t the exact bin averages of t^j
//   1, t_c, t_c^2 + d^2/3, t_c^3 + t_c d^2   (d = h / (2 t_scale)),
// for the exponential exp(b0 + b1 t) its exact average E_c S(b1 d) with
// E_c = exp(b0 + b1 t_c) and S(u) = sinh(u)/u (d/db1 = E_c (t_c S + d S')).
// Each bin evaluates erf and exp at its right edge and hands them to the next
// bin (a thread walking uniform bins edge to edge, or a wave taking 64 bins of
// any widths side by side), so a bin costs one erf and one exp per Gaussian.
// On bins narrower than a sixteenth of every width, the Gaussians' averages
// and partials come instead from a Hermite series about the bin centre, on
// uniform bins with exp at the centres by the two-multiply recurrence (no
// erf; see k_nll_1d_avg).  The objective terms, the
// reverse sweep (w ubar times the partials above) and the reduction are the
// centre model's.  FP64 only.
#pragma once

#include <type_traits>

#include "chunk.hpp"
#include "nll_kernels.hpp"

namespace hf {

// Bins per thread per step of the bin-average kernel.
constexpr int kAvgChunk = 8;

// Terms of the bin-average Hermite series (see k_nll_1d_avg): at most 7.
constexpr int kHermMax = 6;

// sum_{k<=NH} He_2k(z) c_k, sum He_2k+1(z) c_k and sum_{k<=NH} He_2k+2(z) c_k
// (He by He_{n+1} = z He_n - n He_{n-1}).
template <int NH>
__device__ __forceinline__ void herm_series(double z, const double (&c)[kHermMax + 1], double& sv,
                                            double& tv, double& ux) {
  double hm = 1.0, hc = z;
  sv = c[0];
  tv = c[0] * z;
  ux = 0.0;
#pragma unroll
  for (int n = 1; n <= 2 * NH + 1; ++n) {
    const double hn = fma(z, hc, -static_cast<double>(n) * hm);  // He_{n+1}
    hm = hc;
    hc = hn;
    const int m = n + 1;
    if (m % 2 == 0) {
      if (m / 2 <= NH) sv = fma(c[m / 2], hn, sv);
      ux = fma(c[m / 2 - 1], hn, ux);
    } else if ((m - 1) / 2 <= NH) {
      tv = fma(c[(m - 1) / 2], hn, tv);
    }
  }
}

// Uniform bins.  a.x0 holds the left edge of bin 0 (not its centre).
template <int NG, int BKG, int OBJ, bool GRAD>
__global__ __launch_bounds__(kBlock) void k_nll_1d_avg(NllArgs a) {
  using S = Shape1D<NG, BKG>;
  constexpr int P = S::P;
  constexpr int NV = GRAD ? P + 1 : 1;
  constexpr int G1 = NG > 0 ? NG : 1;
  constexpr double kRt = 1.2533141373155002512;   // sqrt(pi/2)
  __shared__ double2 lut[OBJ == OBJ_POISSON ? kLogLut : 1];
  if constexpr (OBJ == OBJ_POISSON) log_lut_load(lut, a.log_lut);
  __shared__ double ec[kErfNear + kErfFar];
  erf_load(ec);
  Model1D<NG, BKG> M;
  M.init(a.theta, a.t_shift, a.t_scale);
  double sg[G1];
#pragma unroll
  for (int g = 0; g < NG; ++g) sg[g] = a.theta[3 * g + 2];
  const double invh = 1.0 / a.hx;
  const double d = 0.5 * a.hx * M.ta;
  // Uniform bins narrow against every width (16 |dz| <= 1, dz = h/s): the
  // Gaussians' bin averages by the Hermite series about the bin centres,
  // with exp at the centres by the two-multiply recurrence, instead of erf at
  // the edges.  With phi(z) = exp(-z^2/2), phi^(n) = (-1)^n He_n phi, so over
  // a bin [z_c - delta, z_c + delta] (delta = dz/2)
  //   avg phi     = phi(z_c) sum_k He_2k(z_c)   c_k,
  //   avg z phi   = phi(z_c) sum_k He_2k+1(z_c) c_k,
  //   avg z^2 phi = phi(z_c) sum_k (He_2k+2 + He_2k)(z_c) c_k,
  // c_k = delta^2k / (2k+1)!, and mu_g = A avg phi, dmu/dm = (A/s) avg z phi,
  // dmu/ds = (A/s) avg z^2 phi.  The first omitted term is at most about
  // (13 delta)^(2N+2)/(2N+3)! relative for |z_c| <= 9 (He_n(z) <= (|z| +
  // sqrt n)^n) and phi < 3e-18 beyond; N = 1, 3 or 6 terms after the first
  // keep it below 1e-19, 1e-19 and 3e-18 for delta up to 4.5e-6, 1.6e-3 and
  // 1/32.
  bool series = NG > 0;
  double dmax = 0.0;
  double dzs[G1], Dz[G1], cs[G1][kHermMax + 1];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    dzs[g] = a.hx * M.is[g];
    series = series && 16.0 * fabs(dzs[g]) <= 1.0;
    dmax = fmax(dmax, 0.5 * fabs(dzs[g]));
    Dz[g] = exp_fast(-dzs[g] * dzs[g]);
    const double d2 = 0.25 * dzs[g] * dzs[g];
    cs[g][0] = 1.0;
#pragma unroll
    for (int k = 1; k <= kHermMax; ++k)
      cs[g][k] = cs[g][k - 1] * d2 / static_cast<double>((2 * k) * (2 * k + 1));
  }
  const int nh = dmax <= 4.5e-6 ? 1 : (dmax <= 1.6e-3 ? 3 : kHermMax);
  __syncthreads();
  double acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  int flags = 0;
  const double seed = (a.grad_w_out && a.seed) ? a.seed[0] : 1.0;  // for grad_w
  const bool finite = all_finite(a.theta, a.P);
  const int64_t nb = a.nx;
  const int64_t nch = (nb + kAvgChunk - 1) / kAvgChunk;
  const int64_t tid = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  for (int64_t c = tid; c < nch; c += stride) {
    const int64_t i0 = c * kAvgChunk;
    const int len = static_cast<int>(nb - i0 < kAvgChunk ? nb - i0 : kAvgChunk);
    // erf path: z, erf and phi at the left edge of the current bin; series
    // path: za = z at the chunk's first centre, ea = phi at the current
    // centre and Ea its ratio to the next one
    double za[G1], Ea[G1], ea[G1];
    if (series) {
      const double xc = fma(static_cast<double>(i0) + 0.5, a.hx, a.x0);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        za[g] = (xc - M.m[g]) * M.is[g];  // z at the first centre
        ea[g] = exp_fast(-0.5 * za[g] * za[g]);
        Ea[g] = exp_fast(fmin(fmax(fma(-dzs[g], za[g], -0.5 * dzs[g] * dzs[g]), -700.0), 700.0));
      }
    } else {
      const double x = fma(static_cast<double>(i0), a.hx, a.x0);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        za[g] = (x - M.m[g]) * M.is[g];
        ea[g] = exp_fast(-0.5 * za[g] * za[g]);
        Ea[g] = erf_from_phi(za[g], ea[g], ec);
      }
    }
    // the next bin's count and weight are requested while the current bin is
    // computed
    double n_nx = load_count1(a, i0);
    double w_nx = a.weights ? static_cast<double>(a.weights[i0]) : 1.0;
    for (int k = 0; k < len; ++k) {
      asm volatile("" ::: "memory");  // the coefficients are read again
      const int64_t i = i0 + k;
      const double n = n_nx, w = w_nx;
      const double xb = fma(static_cast<double>(i + 1), a.hx, a.x0);
      if (k + 1 < len) {
        n_nx = load_count1(a, i + 1);
        w_nx = a.weights ? static_cast<double>(a.weights[i + 1]) : 1.0;
      }
      const double ih = invh;
      double mu = 0.0;
      double J[P];
      if (series) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const double z = fma(static_cast<double>(k), dzs[g], za[g]);  // centre
          double sv, tv, ux;
          if (nh == 1)
            herm_series<1>(z, cs[g], sv, tv, ux);
          else if (nh == 3)
            herm_series<3>(z, cs[g], sv, tv, ux);
          else
            herm_series<kHermMax>(z, cs[g], sv, tv, ux);
          const double es = ea[g] * sv;
          const double mg = M.A[g] * es;
          mu += mg;
          if constexpr (GRAD) {
            const double ae = M.A[g] * M.is[g] * ea[g];
            J[3 * g] = es;
            J[3 * g + 1] = ae * tv;
            J[3 * g + 2] = ae * (sv + ux);
          }
          ea[g] *= Ea[g];  // phi at the next centre
          Ea[g] *= Dz[g];
        }
      } else {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const double zb = (xb - M.m[g]) * M.is[g];
          const double eb = exp_fast(-0.5 * zb * zb);
          const double Eb = erf_from_phi(zb, eb, ec);
          const double ia = sg[g] * kRt * (Eb - Ea[g]) * ih;
          const double mg = M.A[g] * ia;
          mu += mg;
          if constexpr (GRAD) {
            J[3 * g] = ia;
            J[3 * g + 1] = M.A[g] * (ea[g] - eb) * ih;
            J[3 * g + 2] = fma(mg, M.is[g], M.A[g] * fma(za[g], ea[g], -zb * eb) * ih);
          }
          za[g] = zb;
          Ea[g] = Eb;
          ea[g] = eb;
        }
      }
      if constexpr (BKG == BKG_EXP) {
        const double xc = fma(static_cast<double>(i) + 0.5, a.hx, a.x0);
        const double tc = (xc - M.tshift) * M.ta;
        const double dh = d;
        const double Ec = exp_fast(fma(M.c[1], tc, M.c[0]));
        double Sh, dSh;
        sinhc(M.c[1] * dh, Sh, dSh);
        const double eb = Ec * Sh;
        mu += eb;
        if constexpr (GRAD) {
          J[3 * NG] = eb;
          J[3 * NG + 1] = Ec * fma(tc, Sh, dh * dSh);
        }
      } else if constexpr (S::NB > 0) {
        const double xc = fma(static_cast<double>(i) + 0.5, a.hx, a.x0);
        const double tc = (xc - M.tshift) * M.ta;
        const double dh = d;
        const double d2 = dh * dh;
        double avg[4];
        avg[0] = 1.0;
        avg[1] = tc;
        avg[2] = fma(tc, tc, d2 * (1.0 / 3.0));
        avg[3] = tc * fma(tc, tc, d2);
#pragma unroll
        for (int j = 0; j < S::NB; ++j) {
          mu = fma(M.c[j], avg[j], mu);
          if constexpr (GRAD) J[3 * NG + j] = avg[j];
        }
      }
      double l, ub;
      flags |= objective_t<OBJ, false>(n, mu, lut, l, ub) ? ST_DOMAIN : 0;
      acc[0] = fma(w, l, acc[0]);
      if constexpr (GRAD) {
        const double mb = w * ub;
#pragma unroll
        for (int p = 0; p < P; ++p) acc[1 + p] = fma(mb, J[p], acc[1 + p]);
      }
      if (a.grad_w_out) a.grad_w_out[i] = static_cast<float>(seed * l);
    }
  }
  // exact partials: no final factors
  publish_objective<NV>(a, acc, flags | (finite ? 0 : ST_NONFINITE), nullptr, output_seed(a));
}

// x of the lane before, `first` in lane 0.
__device__ __forceinline__ double from_previous_lane(double x, double first) {
  constexpr int kWaveShr1 = 0x138;
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(first), __double2loint(x), kWaveShr1, 0xf,
                                             0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(first), __double2hiint(x), kWaveShr1, 0xf,
                                             0xf, false);
  return __hiloint2double(hi, lo);
}

// Bins of any widths.  A wave takes 64 neighbouring bins per step.
// Where all of them are narrow against every Gaussian's width (h <= s / 16),
// the averages come from the series about the bins' centres that
// k_nll_1d_avg explains, with 2, 3 or 6 terms after the first by the widest
// bin of the step (2 keep the first omitted term below 1e-19 for half-widths
// up to 2.1e-4 s).  It needs no erf, no division and no neighbour, and has
// none of the cancellation of an erf difference over a narrow bin.
// Elsewhere each lane evaluates erf and exp at its bin's right edge; the left
// edge's values come from the lane before by a DPP move, and lane 0's from the
// last lane of the step before.  So loads are contiguous and a bin costs one
// erf and exp per Gaussian.
// Bound: VALU issue, about 240 instructions per bin.  Two Gaussians and a
// line, Poisson, on the GPU with the finishing kernel: a thread walking 8 bins
// edge to edge with the library's erf 20.4 us for 1e6 bins and 61.3 for 4e6;
// 64 bins per wave with erf 19.0 and 58.4; with the series 15.4 and 43.3, and
// 15.2 and 38.9 without constants held in registers (build.py, NO_HOIST).
// 1003 bins 14.9, 7.4 and 7.6.  Two steps side by side gain nothing (15.9 and
// 45.6 with 244 registers).
template <int NG, int BKG, int OBJ, bool GRAD>
__global__ __launch_bounds__(kBlock) void k_nll_1d_avg_edges(NllArgs a) {
  using S = Shape1D<NG, BKG>;
  constexpr int P = S::P;
  constexpr int NV = GRAD ? P + 1 : 1;
  constexpr int G1 = NG > 0 ? NG : 1;
  constexpr double kRt = 1.2533141373155002512;   // sqrt(pi/2)
  __shared__ double2 lut[OBJ == OBJ_POISSON ? kLogLut : 1];
  if constexpr (OBJ == OBJ_POISSON) log_lut_load(lut, a.log_lut);
  __shared__ double ec[kErfNear + kErfFar];
  erf_load(ec);
  Model1D<NG, BKG> M;
  M.init(a.theta, a.t_shift, a.t_scale);
  double sg[G1];
#pragma unroll
  for (int g = 0; g < NG; ++g) sg[g] = a.theta[3 * g + 2];
  __syncthreads();
  double acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  int flags = 0;
  const double seed = (a.grad_w_out && a.seed) ? a.seed[0] : 1.0;  // for grad_w
  const bool finite = all_finite(a.theta, a.P);
  const double* __restrict__ E = a.x_edges;
  const int64_t nb = a.nx;
  const int64_t steps = (nb + 63) / 64;
  const int64_t waves = static_cast<int64_t>(gridDim.x) * kWaves;
  const int64_t wave = static_cast<int64_t>(blockIdx.x) * kWaves + (threadIdx.x >> 6);
  const int lane = static_cast<int>(threadIdx.x & 63u);
  const int64_t s0 = steps * wave / waves, s1 = steps * (wave + 1) / waves;
  if (s0 < s1) {
    // ms: the means for the series' polynomials, no more than 64 widths outside
    // the histogram: farther away phi is 0 (from 39 on), which only finite
    // polynomials leave so
    double us[G1], ms[G1], ismax = 0.0;
    const double e_lo = E[0], e_hi = E[nb];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      us[g] = gauss_unit(M.is[g], sg[g]);
      ismax = fmax(ismax, fabs(M.is[g]));
      const double far = 64.0 * fabs(sg[g]);
      ms[g] = fmin(fmax(M.m[g], e_lo - far), e_hi + far);
    }
    // z, erf and phi at an edge
    struct Edge {
      double z[G1], E[G1], e[G1];
    };
    auto edge = [&](double x) {
      Edge r;
      double u[G1];
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        r.z[g] = (x - M.m[g]) * M.is[g];
        u[g] = (x - M.m[g]) * us[g];
      }
      if constexpr (NG > 0) gauss_n(u, r.e);
#pragma unroll
      for (int g = 0; g < NG; ++g) r.E[g] = erf_from_phi(r.z[g], r.e[g], ec);
      return r;
    };
    double x_last = E[64 * s0];  // right edge of the bin before the step
    Edge last;                   // and its values, where last_set
    bool last_set = false;
    auto bin = [&](int64_t s) {
      const int64_t i = 64 * s + lane;
      return i < nb ? i : nb - 1;
    };
    int64_t i_nx = bin(s0);
    double x_nx = E[i_nx + 1], n_nx = load_count1(a, i_nx);
    double w_nx = a.weights ? static_cast<double>(a.weights[i_nx]) : 1.0;
    for (int64_t s = s0; s < s1; ++s) {
      const int64_t i = i_nx;
      const bool in = 64 * s + lane < nb;  // lanes past the last bin compute it again and are dropped
      const double n = n_nx, w = w_nx, xb = x_nx;
      if (s + 1 < s1) {
        i_nx = bin(s + 1);
        x_nx = E[i_nx + 1];
        n_nx = load_count1(a, i_nx);
        w_nx = a.weights ? static_cast<double>(a.weights[i_nx]) : 1.0;
      }
      const double x_first = x_last, xa = from_previous_lane(xb, x_last);
      x_last = readlane_d(xb, 63);
      const double h = xb - xa, xc = 0.5 * (xa + xb);
      double mu = 0.0;
      double J[P];
      // the series about the centre (see k_nll_1d_avg)
      auto series = [&](auto terms) {
        constexpr int NH = decltype(terms)::value;
        double u[G1], e[G1];
#pragma unroll
        for (int g = 0; g < NG; ++g) u[g] = (xc - M.m[g]) * us[g];
        if constexpr (NG > 0) gauss_n(u, e);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const double z = (xc - ms[g]) * M.is[g], d = 0.5 * h * M.is[g], d2 = d * d;
          double c[kHermMax + 1];
          c[0] = 1.0;
#pragma unroll
          for (int k = 1; k <= NH; ++k)
            c[k] = c[k - 1] * (d2 * (1.0 / static_cast<double>((2 * k) * (2 * k + 1))));
          double sv, tv, ux;
          herm_series<NH>(z, c, sv, tv, ux);
          const double es = e[g] * sv;
          mu = fma(M.A[g], es, mu);
          if constexpr (GRAD) {
            const double ae = M.A[g] * M.is[g] * e[g];
            J[3 * g] = es;
            J[3 * g + 1] = ae * tv;
            J[3 * g + 2] = ae * (sv + ux);
          }
        }
      };
      const double dmax = 0.5 * fabs(h) * ismax;
      // (an empty bin, or an edge or width that is no number: as the erf says)
      const bool small = NG > 0 && __all(!in || (h != 0.0 && dmax <= 1.0 / 32.0));
      if (small) {
        last_set = false;
        if (__all(!in || dmax <= 2.1e-4))
          series(std::integral_constant<int, 2>{});
        else if (__all(!in || dmax <= 1.6e-3))
          series(std::integral_constant<int, 3>{});
        else
          series(std::integral_constant<int, kHermMax>{});
      } else {
        asm volatile("" ::: "memory");  // the coefficients are read again
        if (!last_set) last = edge(x_first);
        last_set = true;
        const Edge right = edge(xb);
        const double ih = in ? 1.0 / h : 0.0;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const double Ea = from_previous_lane(right.E[g], last.E[g]);
          const double ia = sg[g] * kRt * (right.E[g] - Ea) * ih;
          const double mg = M.A[g] * ia;
          mu = fma(M.A[g], ia, mu);
          if constexpr (GRAD) {
            const double za = from_previous_lane(right.z[g], last.z[g]);
            const double ea = from_previous_lane(right.e[g], last.e[g]);
            J[3 * g] = ia;
            J[3 * g + 1] = M.A[g] * (ea - right.e[g]) * ih;
            J[3 * g + 2] = fma(mg, M.is[g], M.A[g] * fma(za, ea, -right.z[g] * right.e[g]) * ih);
          }
        }
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          last.z[g] = readlane_d(right.z[g], 63);
          last.E[g] = readlane_d(right.E[g], 63);
          last.e[g] = readlane_d(right.e[g], 63);
        }
      }
      const double tc = (xc - M.tshift) * M.ta;
      const double dh = 0.5 * h * M.ta;
      if constexpr (BKG == BKG_EXP) {
        const double Ec = exp_fast(fma(M.c[1], tc, M.c[0]));
        double Sh, dSh;
        sinhc(M.c[1] * dh, Sh, dSh);
        const double eb = Ec * Sh;
        mu = fma(Ec, Sh, mu);
        if constexpr (GRAD) {
          J[3 * NG] = eb;
          J[3 * NG + 1] = Ec * fma(tc, Sh, dh * dSh);
        }
      } else if constexpr (S::NB > 0) {
        const double d2 = dh * dh;
        double avg[4];
        avg[0] = 1.0;
        avg[1] = tc;
        avg[2] = fma(tc, tc, d2 * (1.0 / 3.0));
        avg[3] = tc * fma(tc, tc, d2);
#pragma unroll
        for (int j = 0; j < S::NB; ++j) {
          mu = fma(M.c[j], avg[j], mu);
          if constexpr (GRAD) J[3 * NG + j] = avg[j];
        }
      }
      double l, ub;
      const bool dom = objective_t<OBJ, false>(n, mu, lut, l, ub);
      if (in) {
        flags |= dom ? ST_DOMAIN : 0;
        acc[0] = fma(w, l, acc[0]);
        if constexpr (GRAD) {
          const double mb = w * ub;
#pragma unroll
          for (int p = 0; p < P; ++p) acc[1 + p] = fma(mb, J[p], acc[1 + p]);
        }
        if (a.grad_w_out) a.grad_w_out[i] = static_cast<float>(seed * l);
      }
    }
  }
  // exact partials: no final factors
  publish_objective<NV>(a, acc, flags | (finite ? 0 : ST_NONFINITE), nullptr, output_seed(a));
}

// Centre model on bins of any widths: mu at each bin's midpoint, with the
// closed-form partials (A: e; m: G z; s: G z^2, the 1/s applied to the
// totals; polynomial t^j; exponential E and t E), one exp per Gaussian.
// A thread takes kEdgeChunk consecutive bins per step (their kEdgeChunk + 1
// edges are shared between neighbours), their exponentials in step, and
// requests the next step's edges, counts and weights while the current step
// is computed.  Two Gaussians and a line, Poisson, 4e6 bins: 28.5 us on the
// GPU, with one exponential after the other 30.6 (1e6: 12.2 and 13.1).
constexpr int kEdgeChunk = 4;

struct EdgeChunk {
  double e[kEdgeChunk + 1], n[kEdgeChunk], w[kEdgeChunk];
};

__device__ __forceinline__ void load_edge_chunk(const NllArgs& a, int64_t i0, int len,
                                                EdgeChunk& c) {
#pragma unroll
  for (int k = 0; k <= kEdgeChunk; ++k) c.e[k] = k <= len ? a.x_edges[i0 + k] : 0.0;
#pragma unroll
  for (int k = 0; k < kEdgeChunk; ++k) {
    c.n[k] = k < len ? load_count1(a, i0 + k) : 0.0;
    c.w[k] = (k < len && a.weights) ? static_cast<double>(a.weights[i0 + k]) : (k < len ? 1.0 : 0.0);
  }
}

template <int NG, int BKG, int OBJ, bool GRAD>
__global__ __launch_bounds__(kBlock) void k_nll_1d_edges(NllArgs a) {
  using S = Shape1D<NG, BKG>;
  constexpr int P = S::P;
  constexpr int NV = GRAD ? P + 1 : 1;
  constexpr int K = kEdgeChunk;
  __shared__ double2 lut[OBJ == OBJ_POISSON ? kLogLut : 1];
  if constexpr (OBJ == OBJ_POISSON) log_lut_load(lut, a.log_lut);
  Model1D<NG, BKG> M;
  M.init(a.theta, a.t_shift, a.t_scale);
  double us[NG > 0 ? NG : 1];
#pragma unroll
  for (int g = 0; g < NG; ++g) us[g] = gauss_unit(M.is[g], a.theta[3 * g + 2]);
  if constexpr (OBJ == OBJ_POISSON) __syncthreads();
  double acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  int flags = 0;
  const double seed = (a.grad_w_out && a.seed) ? a.seed[0] : 1.0;  // for grad_w
  const bool finite = all_finite(a.theta, a.P);
  const int64_t nb = a.nx;
  const int64_t nch = (nb + K - 1) / K;
  const int64_t tid = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
  EdgeChunk nxt;
  if (tid < nch) {
    const int64_t i0 = tid * K;
    load_edge_chunk(a, i0, static_cast<int>(nb - i0 < K ? nb - i0 : K), nxt);
  }
  for (int64_t c = tid; c < nch; c += stride) {
    const EdgeChunk cur = nxt;
    const int64_t i0 = c * K;
    const int len = static_cast<int>(nb - i0 < K ? nb - i0 : K);
    if (c + stride < nch) {
      const int64_t j0 = (c + stride) * K;
      load_edge_chunk(a, j0, static_cast<int>(nb - j0 < K ? nb - j0 : K), nxt);
    }
    // bins past len (the last chunk) are computed at a valid point and
    // masked: their weight is 0 and their terms are dropped
    double xk[K], u[NG > 0 ? NG * K : 1], ek[NG > 0 ? NG * K : 1];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      xk[k] = k < len ? 0.5 * (cur.e[k] + cur.e[k + 1]) : cur.e[0];
#pragma unroll
      for (int g = 0; g < NG; ++g) u[NG * k + g] = (xk[k] - M.m[g]) * us[g];
    }
    if constexpr (NG > 0) gauss_n(u, ek);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const bool in = k < len;
      const double x = xk[k];
      double mu = 0.0;
      double J[P];
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const double e = ek[NG * k + g], uk = u[NG * k + g];
        mu = fma(M.A[g], e, mu);
        if constexpr (GRAD) {  // the amplitude and the width: on the totals
          J[3 * g] = e;
          J[3 * g + 1] = e * uk;
          J[3 * g + 2] = e * uk * uk;
        }
      }
      const double t = (x - M.tshift) * M.ta;
      if constexpr (BKG == BKG_EXP) {
        const double Eb = exp_fast(fma(M.c[1], t, M.c[0]));
        mu += Eb;
        if constexpr (GRAD) {
          J[3 * NG] = Eb;
          J[3 * NG + 1] = t * Eb;
        }
      } else if constexpr (S::NB > 0) {
        double b = M.c[S::NB - 1];
#pragma unroll
        for (int j = S::NB - 2; j >= 0; --j) b = fma(b, t, M.c[j]);
        mu += b;
        if constexpr (GRAD) {
          double tj = 1.0;
#pragma unroll
          for (int j = 0; j < S::NB; ++j) {
            J[3 * NG + j] = tj;
            tj *= t;
          }
        }
      }
      double l, ub;
      const bool dom = objective_t<OBJ, false>(cur.n[k], mu, lut, l, ub);
      flags |= (dom && in) ? ST_DOMAIN : 0;
      l = in ? l : 0.0;
      acc[0] = fma(cur.w[k], l, acc[0]);
      if constexpr (GRAD) {
        const double mb = in ? cur.w[k] * ub : 0.0;
#pragma unroll
        for (int p = 0; p < P; ++p) acc[1 + p] = fma(mb, J[p], acc[1 + p]);
      }
      if (in && a.grad_w_out) a.grad_w_out[i0 + k] = static_cast<float>(seed * l);
    }
  }
  __shared__ double fac[NV];
  if (threadIdx.x < NV) fac[threadIdx.x] = gauss_factor(M, us, threadIdx.x);
  publish_objective<NV>(a, acc, flags | (finite ? 0 : ST_NONFINITE), fac, output_seed(a));
}

template <int NG, int BKG, int OBJ, bool GRAD>
hipError_t launch_1d_edges(const NllArgs& a, int grid, hipStream_t s, int* occ, int* block) {
  return launch_or_occupancy<kBlock>(k_nll_1d_edges<NG, BKG, OBJ, GRAD>, a, grid, s, occ, block);
}

template <int NG, int BKG>
LaunchFn pick_edges_obj(int obj, bool grad) {
  switch (obj) {
    case OBJ_NEYMAN:
      return grad ? &launch_1d_edges<NG, BKG, OBJ_NEYMAN, true>
                  : &launch_1d_edges<NG, BKG, OBJ_NEYMAN, false>;
    case OBJ_PEARSON:
      return grad ? &launch_1d_edges<NG, BKG, OBJ_PEARSON, true>
                  : &launch_1d_edges<NG, BKG, OBJ_PEARSON, false>;
    case OBJ_POISSON:
      return grad ? &launch_1d_edges<NG, BKG, OBJ_POISSON, true>
                  : &launch_1d_edges<NG, BKG, OBJ_POISSON, false>;
    default:
      return nullptr;
  }
}

template <int NG>
LaunchFn pick_edges_ng(int bkg, int obj, bool grad) {
  switch (bkg) {
    case BKG_NONE:
      if constexpr (NG == 0) return nullptr;
      else return pick_edges_obj<NG, BKG_NONE>(obj, grad);
    case 0:
      return pick_edges_obj<NG, 0>(obj, grad);
    case 1:
      return pick_edges_obj<NG, 1>(obj, grad);
    case 2:
      return pick_edges_obj<NG, 2>(obj, grad);
    case 3:
      return pick_edges_obj<NG, 3>(obj, grad);
    case BKG_EXP:
      return pick_edges_obj<NG, BKG_EXP>(obj, grad);
    default:
      return nullptr;
  }
}

template <int NG, int BKG, int OBJ, bool GRAD, bool EDGES>
hipError_t launch_1d_avg(const NllArgs& a, int grid, hipStream_t s, int* occ, int* block) {
  if constexpr (EDGES) {
    // the value alone takes the gradient's grid, for the same sums
    if (grid <= 0)
      return launch_or_occupancy<kBlock>(k_nll_1d_avg_edges<NG, BKG, OBJ, true>, a, grid, s, occ, block);
    return launch_or_occupancy<kBlock>(k_nll_1d_avg_edges<NG, BKG, OBJ, GRAD>, a, grid, s, occ, block);
  } else
    return launch_or_occupancy<kBlock>(k_nll_1d_avg<NG, BKG, OBJ, GRAD>, a, grid, s, occ, block);
}

template <int NG, int BKG, bool EDGES>
LaunchFn pick_avg_obj_e(int obj, bool grad) {
  switch (obj) {
    case OBJ_NEYMAN:
      return grad ? &launch_1d_avg<NG, BKG, OBJ_NEYMAN, true, EDGES>
                  : &launch_1d_avg<NG, BKG, OBJ_NEYMAN, false, EDGES>;
    case OBJ_PEARSON:
      return grad ? &launch_1d_avg<NG, BKG, OBJ_PEARSON, true, EDGES>
                  : &launch_1d_avg<NG, BKG, OBJ_PEARSON, false, EDGES>;
    case OBJ_POISSON:
      return grad ? &launch_1d_avg<NG, BKG, OBJ_POISSON, true, EDGES>
                  : &launch_1d_avg<NG, BKG, OBJ_POISSON, false, EDGES>;
    default:
      return nullptr;
  }
}

template <int NG, int BKG>
LaunchFn pick_avg_obj(int obj, bool grad, bool edges) {
  return edges ? pick_avg_obj_e<NG, BKG, true>(obj, grad) : pick_avg_obj_e<NG, BKG, false>(obj, grad);
}

// bkg: the background code (polynomial degree -1..3, or BKG_EXP).
template <int NG>
LaunchFn pick_avg_ng(int bkg, int obj, bool grad, bool edges) {
  switch (bkg) {
    case -1:
      if constexpr (NG == 0) return nullptr;
      else return pick_avg_obj<NG, BKG_NONE>(obj, grad, edges);
    case 0:
      return pick_avg_obj<NG, 0>(obj, grad, edges);
    case 1:
      return pick_avg_obj<NG, 1>(obj, grad, edges);
    case 2:
      return pick_avg_obj<NG, 2>(obj, grad, edges);
    case 3:
      return pick_avg_obj<NG, 3>(obj, grad, edges);
    case BKG_EXP:
      return pick_avg_obj<NG, BKG_EXP>(obj, grad, edges);
    default:
      return nullptr;
  }
}

// Defined in nll1d_avg_ng{0..4}.hip.
LaunchFn pick_edges_ng0(int bkg, int obj, bool grad);
LaunchFn pick_edges_ng1(int bkg, int obj, bool grad);
LaunchFn pick_edges_ng2(int bkg, int obj, bool grad);
LaunchFn pick_edges_ng3(int bkg, int obj, bool grad);
LaunchFn pick_edges_ng4(int bkg, int obj, bool grad);
LaunchFn pick_avg_ng0(int bkg, int obj, bool grad, bool edges);
LaunchFn pick_avg_ng1(int bkg, int obj, bool grad, bool edges);
LaunchFn pick_avg_ng2(int bkg, int obj, bool grad, bool edges);
LaunchFn pick_avg_ng3(int bkg, int obj, bool grad, bool edges);
LaunchFn pick_avg_ng4(int bkg, int obj, bool grad, bool edges);

}  // namespace hf
