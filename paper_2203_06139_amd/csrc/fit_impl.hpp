// fit_impl.hpp -- persistent batched BFGS fitter (templates).
//
// Algorithm per histogram (the optimiser step of a gradient-based fit, paper
// sec. 4; BFGS and the first-step scaling follow Nocedal & Wright,
// "Numerical Optimization", ch. 6 and eq. 6.20):
//   scaled coordinates u_k = (theta_k - theta0_k)/sigma_k for the free
//   parameters, sigma by parameter kind (amplitude max(|A0|,1), mean
//   range/100, width |s0|, background max(|c0|,1));  H = I, or with the
//   Fisher start H = inverse expected Hessian at theta0 (Gauss-Newton /
//   Fisher scoring first step; identity if it is not safely positive
//   definite);
//   repeat: p = -H g;  EDM = g^T H g / 2;  stop when EDM < max(edm_tol,
//   4 eps |f|);  if g^T p >= 0 restart from H = I;  backtracking Armijo
//   (c1 = 1e-4, alpha halved up to ls_max times; non-finite f rejected);
//   s = alpha p, y = g_new - g;  if s^T y > 1e-12 |s||y| the BFGS inverse
//   update (scaled by s^T y / y^T y before the first one after an identity
//   start).
// Finally |s| for every width, Gaussians ordered by mean, and the NLL
// re-evaluated with FP64 bins.
//
// Work split: the whole workgroup (or, for small histograms, one wave)
// evaluates the objective and gradient over the histogram's bins (run_1d, or
// chunk_1d for FP32 bins, then a fixed-order group sum); the group's first
// wave runs the optimiser alone: the O(P^2) algebra is spread over its lanes,
// scalar decisions are computed redundantly by every lane from the same LDS
// values, and the other waves wait for the next point at a barrier.  With the
// whole workgroup in the algebra, each step behind a workgroup barrier, one
// evaluation and iteration of a 256-bin histogram took 3.4 us, 2.9 now (and
// the other waves' issue slots go to the CU's second workgroup: 4096 uneven
// fits 1.12 -> 1.09 ms).
#pragma once

#include <float.h>
#include <type_traits>
#include <stdlib.h>

#include "chunk.hpp"
#include "device.hpp"
#include "fit_kernels.hpp"

namespace hf {

enum : int { FIT_CONVERGED = 0, FIT_MAXITER = 1, FIT_LSFAIL = 2, FIT_NONFINITE = 3,
             FIT_DOMAIN = 4, FIT_BADHIST = 5 };

__device__ __forceinline__ double count_at(const void* base, int dtype, int64_t i) {
  if (dtype == DT_U32) return static_cast<const uint32_t*>(base)[i];
  if (dtype == DT_F32) return static_cast<const float*>(base)[i];
  return static_cast<const double*>(base)[i];
}

// Entries of the expected Hessian summed over the group at a time.
constexpr int kFisherPass = 32;

template <int NG, int BKG, int BLK>
struct FitShared {
  static constexpr int P = Shape1D<NG, BKG>::P;
  static constexpr int NV = P + 1;
  double th[P], th0[P], sig[P];
  double u[P], g[P], un[P], gn[P], pv[P], up[P];
  double H[P * P];   // row stride P; the leading nf x nf block is used
  double tot[NV];
  double red[BLK / 64][NV];
  double fred[(BLK / 64) * kFisherPass];
  int redf[BLK / 64];
  int fredf[BLK / 64];
  int fidx[P];
  int nf;
  int h;
  // the optimiser's state, kept by the group's first wave
  double f, fn, nll, edm, goal, slope, alpha, fp, hp, hm;
  int nev, it, ls, q, status, stage, after, f32, first;
  int cmd;  // what the group evaluates next
};

// Bins per thread per step of the FP32-bin sweep: 8 once every thread of a
// workgroup has a chunk of 8, else 4.  Measured on the
// 4096-histogram Gauss + exponential batch (512-thread workgroups, counts
// in LDS): one evaluation of its longest fit (22,086 bins) 15.2 us with
// 4-bin chunks, 13.5 with 8 and 15.5 with 16; reading the cached counts as
// 16-byte vectors instead of one by one, 12.1 us with 8.
constexpr int kFitChunkSmall = 4;
constexpr int kFitChunkLarge = 8;
// The 8-bin sweep is built where it fits the register budget: 512-thread
// workgroups (two waves per SIMD by construction) of one Gaussian with no,
// a constant or an exponential background, which stay below 256 VGPRs
// without spilling.  With a sloped polynomial background the 8-bin sweep
// spilled at 512 threads (32-144 bytes per lane), and at 256 threads it
// took several models to one wave per SIMD (256 VGPRs plus AGPRs), e.g.
// Gauss + line, Poisson: 0.35 -> 0.46 ms for 512 histograms of 10,000 bins.
template <int NG, int BKG, int BLK>
constexpr bool fit_chunk_large() {
  return BLK == 512 && NG == 1 && (BKG == BKG_NONE || BKG == 0 || BKG == BKG_EXP);
}

// Where a histogram's counts are read from: the workgroup's LDS cache (u32)
// or global memory (any dtype).
struct CountsSrc {
  const uint32_t* lds;  // non-null when cached (16-byte aligned)
  const void* glb;
  int dtype;
  int64_t off;
  __device__ __forceinline__ double at(int64_t i) const {
    return lds ? static_cast<double>(lds[i]) : count_at(glb, dtype, off + i);
  }
  // K consecutive counts from bin i0 (K and i0 multiples of 4)
  template <int K>
  __device__ __forceinline__ void chunk(int64_t i0, double (&n)[K]) const {
    if (lds) {
#pragma unroll
      for (int q = 0; q < K / 4; ++q) {
        const uint4 v = reinterpret_cast<const uint4*>(lds + i0)[q];
        n[4 * q] = v.x;
        n[4 * q + 1] = v.y;
        n[4 * q + 2] = v.z;
        n[4 * q + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) n[k] = count_at(glb, dtype, off + i0 + k);
    }
  }
};

// A thread's groups of four counts in the order run_1d takes them: runs of S
// groups, the threads' runs interleaved.  Counts of u32 type are requested
// one group ahead, into the registers that the group before has just left, so
// a group covers the latency of the next; the index is clamped instead of
// tested, which keeps the loop free of branches.  Where they are read from is
// a template argument for the same reason.
enum : int { SRC_LDS = 0, SRC_U32 = 1, SRC_ANY = 2 };

template <int KIND>
struct RunCounts {
  const CountsSrc& src;
  int q, last, skip, S, left;  // group requested; last group; from a run's end to the next run
  uint4 raw;

  __device__ __forceinline__ RunCounts(const CountsSrc& s, int first, int groups, int per_run,
                                       int threads)
      : src(s), q(first * per_run), last(groups - 1), skip((threads - 1) * per_run), S(per_run),
        left(per_run), raw() {
    request();
  }
  __device__ __forceinline__ void request() {
    // a histogram starts anywhere in the batch: aligned to its values only
    typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));
    const int g = q < last ? q : last;
    if constexpr (KIND == SRC_LDS) {
      raw = reinterpret_cast<const uint4*>(src.lds)[g];
    } else if constexpr (KIND == SRC_U32) {
      const u4 v = *reinterpret_cast<const u4*>(static_cast<const uint32_t*>(src.glb) + src.off +
                                                4 * static_cast<int64_t>(g));
      raw = uint4{v.x, v.y, v.z, v.w};
    }
  }
  __device__ __forceinline__ void operator()(double (&n)[4]) {
    if constexpr (KIND == SRC_ANY) {
#pragma unroll
      for (int k = 0; k < 4; ++k) n[k] = src.at(4 * static_cast<int64_t>(q) + k);
    } else {
      n[0] = raw.x;
      n[1] = raw.y;
      n[2] = raw.z;
      n[3] = raw.w;
    }
    ++q;
    if (--left == 0) {
      left = S;
      q += skip;
    }
    request();
  }
};

// The threads that run one fit: the workgroup (BLK = 256 or 512), or one
// wave (BLK = 64) for the small histograms at the end of the longest-first
// queue.  gtid is the thread's index in its group, gsync the group's
// barrier (for a wave: LDS operations stay in program order, so a fence and
// a code-motion barrier are enough).
template <int BLK>
__device__ __forceinline__ int gtid() {
  return BLK == 64 ? static_cast<int>(threadIdx.x & 63u) : static_cast<int>(threadIdx.x);
}

template <int BLK>
__device__ __forceinline__ void gsync() {
  if constexpr (BLK == 64) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// Each wave's sums of v and its flags into red and redf.
template <int NV, int BLK>
__device__ __forceinline__ void wave_totals(const double (&v)[NV], int flags, double (*red)[NV],
                                            int* redf) {
  const int wid = BLK == 64 ? 0 : static_cast<int>(threadIdx.x >> 6);
  wave_sums(v, [&](int k, double x) { red[wid][k] = x; });
  const int f = (__ballot(flags & ST_DOMAIN) ? ST_DOMAIN : 0) |
                (__ballot(flags & ST_NONFINITE) ? ST_NONFINITE : 0);
  if ((threadIdx.x & 63u) == 0) redf[wid] = f;
}

// The group's total of component k, the waves added in order.
template <int NV, int BLK>
__device__ __forceinline__ double add_waves(const double (*red)[NV], const int* redf, int k, int& flags) {
  double x = red[0][k];
  flags = redf[0];
#pragma unroll
  for (int w = 1; w < BLK / 64; ++w) {
    x += red[w][k];
    flags |= redf[w];
  }
  return x;
}

// Totals of an evaluation for the group's first wave: f in sm.tot[0] (+inf on
// a domain error) and dL/dtheta_k in sm.tot[1 + k].  One group barrier.
template <int NG, int BKG, int BLK, int NV>
__device__ __forceinline__ void publish_totals(FitShared<NG, BKG, BLK>& sm, const Model1D<NG, BKG>& M,
                                               double (&acc)[NV], int flags) {
  double(*red)[NV] = reinterpret_cast<double(*)[NV]>(sm.red);
  wave_totals<NV, BLK>(acc, flags, red, sm.redf);
  gsync<BLK>();
  const int k = gtid<BLK>();
  if (k < 64) {
    if (k < NV) {
      int o;
      double x = add_waves<NV, BLK>(red, sm.redf, k, o);
      if (k == 0 && (o & ST_DOMAIN)) x = __builtin_inf();
      sm.tot[k] = k == 0 ? x : x * M.final_factor(k);
    }
    gsync<64>();
  }
}

// Objective (and with GRAD its gradient) of one histogram at sm.th with FP32
// bins, evaluated by the whole group with the chunked sweep (chunk_1d) in
// K-bin chunks.  Leaves f in sm.tot[0] (+inf on a domain error) and
// dL/dtheta_k in sm.tot[1 + k].
template <int NG, int BKG, int OBJ, bool GRAD, int BLK, int K>
__device__ __forceinline__ void wg_eval_k(const FitArgs& a, FitShared<NG, BKG, BLK>& sm,
    const double2* lut, const CountsSrc& src, int64_t nb, double x0, double hx) {
  constexpr int NV = GRAD ? FitShared<NG, BKG, BLK>::NV : 1;
  Model1D<NG, BKG> M;
  M.init(sm.th, a.t_shift, a.t_scale);
  M.init_grid(hx, K);
  double acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  int flags = 0;
  const int64_t nch = nb / K;
  double w[K];
#pragma unroll
  for (int k = 0; k < K; ++k) w[k] = 1.0;
  for (int64_t c = gtid<BLK>(); c < nch; c += BLK) {
    const int64_t i0 = c * K;
    double n[K];
    src.chunk<K>(i0, n);
    double l[K];
    const double xs = fma(static_cast<double>(i0), hx, x0);
    if (M.recur)
      chunk_1d<NG, BKG, OBJ, GRAD, true, true>(M, lut, xs, n, w, acc, flags, l);
    else
      chunk_1d<NG, BKG, OBJ, GRAD, true, false>(M, lut, xs, n, w, acc, flags, l);
  }
  for (int64_t i = nch * K + gtid<BLK>(); i < nb; i += BLK) {
    const double n1[1] = {src.at(i)};
    const double w1[1] = {1.0};
    double l1[1];
    chunk_1d<NG, BKG, OBJ, GRAD, true, false>(M, lut, fma(static_cast<double>(i), hx, x0), n1, w1,
                                                acc, flags, l1);
  }
  publish_totals<NG, BKG, BLK>(sm, M, acc, flags);
}

// Groups of four bins per run of the FP64 sweep: the S <= kRunGroups with
// the least work on the busiest thread, counting a run's start and expansion
// (two exps per Gaussian and the moments) as kRunStart bins.
constexpr int kRunGroups = 8;

// Groups of four bins that are taken in runs; the bins after them are taken
// one by one (at most three, and those beyond 2^31).
__device__ __forceinline__ int run_quads(int64_t nb) {
  return nb < (int64_t(1) << 31) ? static_cast<int>(nb / 4) : (1 << 29) - (1 << 16);
}

template <int NG>
__device__ __forceinline__ int run_groups(int64_t nb, int threads) {
  constexpr unsigned kRunStart = 2 + NG;
  const unsigned n = run_quads(nb);
  int best = 1;
  unsigned cost = ~0u;
#pragma unroll
  for (int S = 1; S <= kRunGroups; ++S) {
    const unsigned runs = (n + S - 1) / S;
    const unsigned c = (runs + threads - 1) / threads * (4 * S + kRunStart);
    if (c < cost) {
      cost = c;
      best = S;
    }
  }
  return best;
}

// The same evaluation in FP64 by runs of S groups of four bins (run_1d), in
// single groups where a run is too long for the recurrences, and in groups
// with an exponential per bin and Gaussian where four bins are.
// Bound: VALU issue, about 43 instructions per bin in runs.  Narrow peaks (1 to
// 3 bins): the four bins' chains side by side, 10,000 bins of one Gaussian and
// a line 71 us a fit, bin by bin 123; 64 of three Gaussians on 100,000 bins
// 1.55 ms and 2.7.
// Against four-bin chunks, each with its own exps and expansion, and counts
// read as they were needed: one evaluation and iteration of a 65,536-bin
// Gauss + exponential histogram on 256 threads 67.5 -> 32 us; 4096 such
// histograms of 256..65536 bins 1.84 -> 1.14 ms; 512 of three Gaussians + line
// on 10,000 bins 0.70 -> 0.33 ms (280 -> 256 registers: two waves per SIMD).
template <int NG, int BKG, int OBJ, bool GRAD, int BLK>
__device__ __forceinline__ void wg_eval_runs(const FitArgs& a, FitShared<NG, BKG, BLK>& sm,
    const double2* lut, const CountsSrc& src, int64_t nb, double x0, double hx, int S) {
  constexpr int NV = GRAD ? FitShared<NG, BKG, BLK>::NV : 1;
  const int tid = gtid<BLK>();
  Model1D<NG, BKG> M;
  M.init_wave(sm.th, a.t_shift, a.t_scale, hx, 4 * S);
  if (!M.recur && S > 1) {
    S = 1;
    M.recur = M.recurs(4);
  }
  double acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = 0.0;
  int flags = 0;
  // with a bin per thread at most, a group of four would leave threads idle
  // (256 narrow bins on 256 threads: 27 us a fit, in groups 29)
  const int nq = M.recur || nb > BLK ? run_quads(nb) : 0;
  auto runs = [&](auto kind) {
    RunCounts<decltype(kind)::value> next(src, tid, nq, S, BLK);
    for (int q = tid * S; q < nq; q += BLK * S)
      run_1d<NG, BKG, OBJ, GRAD>(M, lut, fma(4.0 * q, hx, x0), nq - q < S ? nq - q : S, next, acc, flags);
  };
  auto groups = [&](auto kind) {
    RunCounts<decltype(kind)::value> next(src, tid, nq, 1, BLK);
    const double w4[4] = {1.0, 1.0, 1.0, 1.0};
    for (int q = tid; q < nq; q += BLK) {
      double n4[4], l4[4];
      next(n4);
      chunk_1d<NG, BKG, OBJ, GRAD, false, false>(M, lut, fma(4.0 * q, hx, x0), n4, w4, acc, flags, l4);
    }
  };
  if (nq > 0) {
    if (M.recur) {
      if (src.lds)
        runs(std::integral_constant<int, SRC_LDS>{});
      else if (src.dtype == DT_U32)
        runs(std::integral_constant<int, SRC_U32>{});
      else
        runs(std::integral_constant<int, SRC_ANY>{});
    } else if (!src.lds && src.dtype == DT_U32) {  // (a third kind costs the FP32 sweep 4%)
      groups(std::integral_constant<int, SRC_U32>{});
    } else {
      groups(std::integral_constant<int, SRC_ANY>{});
    }
  }
  const double w1[1] = {1.0};
  for (int64_t i = 4 * static_cast<int64_t>(nq) + tid; i < nb; i += BLK) {
    const double n1[1] = {src.at(i)};
    double l1[1];
    chunk_1d<NG, BKG, OBJ, GRAD, false, false>(M, lut, fma(static_cast<double>(i), hx, x0), n1, w1,
                                               acc, flags, l1);
  }
  publish_totals<NG, BKG, BLK>(sm, M, acc, flags);
}

// S: run_groups() of the histogram.  FP32 bins take their exps per chunk in
// FP32, which is part of their results, and keep the chunked sweep.
template <int NG, int BKG, int OBJ, bool F32BIN, bool GRAD, int BLK>
__device__ __forceinline__ void wg_eval(const FitArgs& a, FitShared<NG, BKG, BLK>& sm,
    const double2* lut, const CountsSrc& src, int64_t nb, double x0, double hx, int S) {
  if constexpr (!F32BIN) {
    wg_eval_runs<NG, BKG, OBJ, GRAD, BLK>(a, sm, lut, src, nb, x0, hx, S);
  } else {
    if constexpr (fit_chunk_large<NG, BKG, BLK>()) {
      if (nb >= static_cast<int64_t>(kFitChunkLarge) * BLK) {
        wg_eval_k<NG, BKG, OBJ, GRAD, BLK, kFitChunkLarge>(a, sm, lut, src, nb, x0, hx);
        return;
      }
    }
    wg_eval_k<NG, BKG, OBJ, GRAD, BLK, kFitChunkSmall>(a, sm, lut, src, nb, x0, hx);
  }
}

// mu(x) and dmu/dtheta by their closed forms, one exp per Gaussian:
//   dG/dA = e, dG/dm = G z / s, dG/ds = G z^2 / s with z = (x - m)/s, the
//   1/s left to Model1D::final_factor; polynomial t^j; exponential E and t E.
template <int NG, int BKG>
__device__ __forceinline__ double mu_partials(const Model1D<NG, BKG>& M, double x,
                                              double (&v)[Shape1D<NG, BKG>::P]) {
  using S = Shape1D<NG, BKG>;
  double mu = 0.0;
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const double z = (x - M.m[g]) * M.is[g];
    const double e = exp_fast(-0.5 * z * z);
    const double G = M.A[g] * e;
    mu += G;
    v[3 * g] = e;
    v[3 * g + 1] = G * z;
    v[3 * g + 2] = G * z * z;
  }
  const double t = (x - M.tshift) * M.ta;
  if constexpr (BKG == BKG_EXP) {
    const double E = exp_fast(fma(M.c[1], t, M.c[0]));
    mu += E;
    v[3 * NG] = E;
    v[3 * NG + 1] = t * E;
  } else if constexpr (S::NB > 0) {
    double tj = 1.0;
#pragma unroll
    for (int j = 0; j < S::NB; ++j) {
      mu = fma(M.c[j], tj, mu);
      v[3 * NG + j] = tj;
      tj *= t;
    }
  }
  return mu;
}

// Weight c of the expected Hessian, 0 where the bin is skipped.
template <int OBJ>
__device__ __forceinline__ double fisher_weight(double n, double mu) {
  if constexpr (OBJ == OBJ_NEYMAN) return n > 0.0 ? 2.0 / n : 0.0;
  return (OBJ == OBJ_PEARSON ? 2.0 : 1.0) / mu;
}

// acc[q] += c v_a v_b for the upper-triangle entries E0 .. E0 + NQ.
template <int P, int E0, int NQ>
__device__ __forceinline__ void fisher_add(double c, const double (&v)[P], double (&acc)[NQ]) {
  constexpr TriIndex<P> tri{};
  if (c > 0.0 && __builtin_isfinite(c)) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = fma(c * v[tri.a[E0 + q]], v[tri.b[E0 + q]], acc[q]);
  }
}

// mu and its partials at four consecutive bins by the recurrences of run_1d,
// z and t from the group's start.
template <int NG, int BKG>
__device__ __forceinline__ void mu_partials_4(const Model1D<NG, BKG>& M, double xs, double (&mu)[4],
                                              double (&v)[4][Shape1D<NG, BKG>::P]) {
  using S = Shape1D<NG, BKG>;
#pragma unroll
  for (int k = 0; k < 4; ++k) mu[k] = 0.0;
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const double z0 = (xs - M.m[g]) * M.is[g];
    double e = exp_fast(-0.5 * z0 * z0);
    double rho = expm1_fast(clamp_ratio_exponent<false>(fma(-M.dz[g], z0, -0.5 * M.dz[g] * M.dz[g])));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double z = fma(static_cast<double>(k), M.dz[g], z0), G = M.A[g] * e;
      mu[k] += G;
      v[k][3 * g] = e;
      v[k][3 * g + 1] = G * z;
      v[k][3 * g + 2] = G * z * z;
      e = fma(e, rho, e);
      rho = fma(-M.Dm[g], rho, rho - M.Dm[g]);
    }
  }
  const double t0 = (xs - M.tshift) * M.ta;
  double E = 0.0;
  if constexpr (BKG == BKG_EXP) E = exp_fast(fma(M.c[1], t0, M.c[0]));
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double t = fma(static_cast<double>(k), M.dt, t0);
    if constexpr (BKG == BKG_EXP) {
      mu[k] += E;
      v[k][3 * NG] = E;
      v[k][3 * NG + 1] = t * E;
      E = fma(E, M.qEm, E);
    } else if constexpr (S::NB > 0) {
      double tj = 1.0;
#pragma unroll
      for (int j = 0; j < S::NB; ++j) {
        mu[k] = fma(M.c[j], tj, mu[k]);
        v[k][3 * NG + j] = tj;
        tj *= t;
      }
    }
  }
}

// Expected Hessian at theta0, F = sum_i c_i (dmu_i/dtheta)(dmu_i/dtheta)^T
// with c_i = d^2 l/d mu^2 at n_i = mu_i (1/mu Poisson, 2/mu Pearson, 2/n for
// n > 0 Neyman); bins whose c_i is not finite and positive are skipped.  The
// upper triangle is accumulated up to kFisherWide entries per pass over the
// bins (one pass for P <= 11, two up to 16), summed over the group
// kFisherPass entries at a time and written symmetrically into sm.H.
// The recurrences run over four bins only: against 64-bit mantissas the
// entries are then as good as with an exponential per bin (10,000 bins of three
// Gaussians: 4.4e-17 of their scale rms, and 4.8e-17), where the runs of an
// evaluation leave 9.5e-17.  4096 fits of 256..65536 bins: 975 us, with an
// exponential per bin 1010, by the runs 945.
constexpr int kFisherWide = 72;
template <int NG, int BKG, int OBJ, int PASS, int BLK>
__device__ __forceinline__ void fisher_pass(const FitArgs& a, FitShared<NG, BKG, BLK>& sm,
    const CountsSrc& src, int64_t nb, double x0, double hx) {
  constexpr int P = FitShared<NG, BKG, BLK>::P;
  constexpr TriIndex<P> tri{};
  constexpr int N = TriIndex<P>::N;
  constexpr int W = (N + (N + kFisherWide - 1) / kFisherWide - 1) / ((N + kFisherWide - 1) / kFisherWide);
  constexpr int E0 = PASS * W;
  if constexpr (E0 < N) {
    constexpr int NQ = (N - E0 < W) ? N - E0 : W;
    const int tid = gtid<BLK>();
    Model1D<NG, BKG> M;
    M.init_wave(sm.th0, a.t_shift, a.t_scale, hx, 4);
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    auto weight = [&](int64_t i, double mu) {  // only Neyman's reads the counts
      return fisher_weight<OBJ>(OBJ == OBJ_NEYMAN ? src.at(i) : 0.0, mu);
    };
    const int64_t nq = M.recur ? nb / 4 : 0;
    for (int64_t q = tid; q < nq; q += BLK) {
      double mu[4], v[4][P];
      mu_partials_4(M, fma(4.0 * static_cast<double>(q), hx, x0), mu, v);
#pragma unroll
      for (int k = 0; k < 4; ++k) fisher_add<P, E0>(weight(4 * q + k, mu[k]), v[k], acc);
    }
    for (int64_t i = 4 * nq + tid; i < nb; i += BLK) {
      double v[P];
      const double mu = mu_partials(M, fma(static_cast<double>(i), hx, x0), v);
      fisher_add<P, E0>(weight(i, mu), v, acc);
    }
#pragma unroll
    for (int c0 = 0; c0 < NQ; c0 += kFisherPass) {
      double part[kFisherPass];
#pragma unroll
      for (int q = 0; q < kFisherPass; ++q) part[q] = c0 + q < NQ ? acc[c0 + q < NQ ? c0 + q : 0] : 0.0;
      double(*red)[kFisherPass] = reinterpret_cast<double(*)[kFisherPass]>(sm.fred);
      wave_totals<kFisherPass, BLK>(part, 0, red, sm.fredf);
      gsync<BLK>();
      if (tid < kFisherPass && c0 + tid < NQ) {
        int o;
        const int r = tri.a[E0 + c0 + tid], c = tri.b[E0 + c0 + tid];
        const double f = add_waves<kFisherPass, BLK>(red, sm.fredf, tid, o) * M.final_factor(1 + r) *
                         M.final_factor(1 + c);
        sm.H[r * P + c] = f;
        sm.H[c * P + r] = f;
      }
      gsync<BLK>();
    }
    fisher_pass<NG, BKG, OBJ, PASS + 1, BLK>(a, sm, src, nb, x0, hx);
  }
}

// Replaces F in sm.H by the inverse of F_u = diag(sigma) F diag(sigma) over
// the free parameters: Cholesky F_u = L L^T (a pivot must exceed 1e-12 times
// the largest diagonal entry), X = inv(L), H = X^T X.  Falls back to the
// identity when F_u is not safely positive definite or anything is not
// finite.  Returns whether the inverse was taken.  One wave: lane r holds row
// r of F_u and L, then column r of X, in registers, and takes the other
// lanes' values by readlane; rows past nf are the identity's.
template <int NG, int BKG, int BLK>
__device__ __forceinline__ bool fisher_start(FitShared<NG, BKG, BLK>& sm, int nf) {
  constexpr int P = FitShared<NG, BKG, BLK>::P;
  const int r = static_cast<int>(threadIdx.x & 63u);
  const bool mine = r < nf;
  const int kr = mine ? sm.fidx[r] : 0;
  const double sr = sm.sig[kr];
  double a[P], x[P];
  double diag = mine ? sr * sr * sm.H[kr * P + kr] : 0.0;
#pragma unroll
  for (int c = 0; c < P; ++c) {
    const int kc = c < nf ? sm.fidx[c] : 0;
    a[c] = mine && c < nf ? sr * sm.sig[kc] * sm.H[kr * P + kc] : (r == c ? 1.0 : 0.0);
  }
  double dmax = 0.0;
#pragma unroll
  for (int c = 0; c < P; ++c) dmax = fmax(dmax, readlane_d(diag, c));
  bool ok = dmax > 0.0 && __builtin_isfinite(dmax);
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const double d = readlane_d(a[j], j);
    if (j < nf && (!(d > 1e-12 * dmax) || !__builtin_isfinite(d))) ok = false;
    const double piv = sqrt(d);
    a[j] = r == j ? piv : a[j] / piv;
#pragma unroll
    for (int c = j + 1; c < P; ++c) a[c] = fma(-a[j], readlane_d(a[j], c), a[c]);
  }
#pragma unroll
  for (int i = 0; i < P; ++i) {
    double v = r == i ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < i; ++k) v = fma(-readlane_d(a[k], i), x[k], v);
    x[i] = v / readlane_d(a[i], i);
  }
  gsync<64>();  // every lane has read F
#pragma unroll
  for (int c = 0; c < P; ++c) {
    double v = 0.0;
#pragma unroll
    for (int k = c; k < P; ++k) v = fma(x[k], readlane_d(x[k], c), v);
    if (mine && c < nf && !__builtin_isfinite(v)) ok = false;
    a[c] = v;
  }
  ok = __all(ok);
  if (r < P) {
#pragma unroll
    for (int c = 0; c < P; ++c) sm.H[r * P + c] = ok && mine && c < nf ? a[c] : (r == c ? 1.0 : 0.0);
  }
  gsync<64>();
  return ok;
}

// Sum over the first 16 lanes, wave-uniform.
__device__ __forceinline__ double lane_sum(double v) { return readlane_d(row_sum(v), 0); }

// Row of H (one per lane) times the vector whose entries the lanes hold: four
// partial sums, so that the chain is P / 4 + 2 operations long.
template <int P>
__device__ __forceinline__ double row_times(const double (&h)[P], double v) {
  double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int c = 0; c < P; ++c) s[c & 3] = fma(h[c], readlane_d(v, c), s[c & 3]);
  return (s[0] + s[1]) + (s[2] + s[3]);
}

// Central differences in the scaled coordinates, the gradient a fitter
// without derivatives of the model uses: g_q = (f(u + h e_q) - f(u - h e_q))
// / (2h) with h = kFdStep max(1, |u_q|), 2 nf objective sweeps.
constexpr double kFdStep = 1e-4;

// What an evaluation was for (optimiser_step), and what is evaluated next.
enum : int { EV_INIT = 0, EV_POLISH, EV_SEARCH, EV_FINAL, EV_FD_PLUS, EV_FD_MINUS };
enum : int { CMD_DONE = 0, CMD_VALUE, CMD_F32, CMD_F64 };

// Sets the group's next evaluation: at the point `un` (or `up` for central
// differences) of the scaled free coordinates.
template <int NG, int BKG, int BLK>
__device__ __forceinline__ void optimiser_point(const FitArgs& a, FitShared<NG, BKG, BLK>& sm, int stage,
                                                bool f32) {
  const int lane = static_cast<int>(threadIdx.x & 63u);
  if (lane < sm.nf) {
    const int k = sm.fidx[lane];
    sm.th[k] = fma(sm.sig[k], stage >= EV_FD_PLUS ? sm.up[lane] : sm.un[lane], sm.th0[k]);
  }
  if (lane == 0) {
    sm.stage = stage;
    sm.f32 = f32 ? 1 : 0;
    sm.cmd = a.fd_grad != 0 ? CMD_VALUE : (f32 && stage != EV_FINAL ? CMD_F32 : CMD_F64);
  }
}

template <int NG, int BKG, int BLK>
__device__ __forceinline__ void optimiser_end(FitShared<NG, BKG, BLK>& sm, double nll, int status) {
  if ((threadIdx.x & 63u) == 0) {
    sm.nll = nll;
    sm.status = status;
    sm.cmd = CMD_DONE;
  }
}

// First Hessian and the evaluation at the start.
template <int NG, int BKG, int OBJ, int BLK>
__device__ __forceinline__ void optimiser_begin(const FitArgs& a, FitShared<NG, BKG, BLK>& sm) {
  constexpr int P = FitShared<NG, BKG, BLK>::P;
  const int lane = static_cast<int>(threadIdx.x & 63u);
  bool first = true;  // scale H at the first update: not after a Fisher start
  if (a.hessian_init == 1 && sm.nf > 0) {
    first = !fisher_start(sm, sm.nf);
  } else {
    for (int t = lane; t < P * P; t += 64) sm.H[t] = (t / P == t % P) ? 1.0 : 0.0;
  }
  if (lane == 0) {
    sm.first = first ? 1 : 0;
    sm.f = sm.edm = sm.goal = sm.slope = 0.0;
    sm.alpha = 1.0;
    sm.nev = 1;
    sm.it = sm.ls = sm.q = 0;
    sm.status = FIT_MAXITER;
  }
  optimiser_point(a, sm, EV_INIT, a.f32 != 0);
}

// Takes the evaluation of sm.tot and sets the next one, or ends the fit.
// Scalar decisions are computed redundantly by every lane from the same LDS
// values, so control flow is uniform.
template <int NG, int BKG, int OBJ, int BLK>
__device__ __forceinline__ void optimiser_step(const FitArgs& a, FitShared<NG, BKG, BLK>& sm) {
  constexpr int P = FitShared<NG, BKG, BLK>::P;
  const int lane = static_cast<int>(threadIdx.x & 63u);
  const int nf = sm.nf, stage = sm.stage;
  const bool fd = a.fd_grad != 0;  // central differences (FP64 bins only)
  const bool f32 = sm.f32 != 0;
  const double fe = sm.tot[0];
  double f = sm.f;
  bool accepted = false;
  if (stage == EV_FINAL) return optimiser_end(sm, fe, sm.status);
  if (stage == EV_FD_PLUS) {
    const double hm = sm.hm;
    const int q = sm.q;
    gsync<64>();
    if (lane == 0) sm.fp = fe;
    if (lane < nf) sm.up[lane] = lane == q ? hm : sm.un[lane];
    return optimiser_point(a, sm, EV_FD_MINUS, false);
  }
  int q = 0;  // next coordinate of the differences, if any
  bool differences = false;
  if (stage == EV_FD_MINUS) {
    q = sm.q;
    const double g = (sm.fp - fe) / (sm.hp - sm.hm);
    accepted = sm.after == EV_SEARCH;
    gsync<64>();
    if (lane == 0) sm.gn[q] = g;
    differences = ++q < nf;
    if (!differences && lane == 0) sm.nev += 2 * nf;
    gsync<64>();
  } else {
    bool go_on;
    if (stage == EV_SEARCH) {
      const double alpha = sm.alpha;
      const int ls = sm.ls + 1;
      go_on = accepted = __builtin_isfinite(fe) && fe <= f + 1e-4 * alpha * sm.slope;
      const double edm = sm.edm, goal = sm.goal;
      gsync<64>();
      if (lane == 0) {
        ++sm.nev;
        if (accepted) ++sm.it;
        sm.ls = ls;
        sm.alpha = 0.5 * alpha;
      }
      if (!accepted && ls < a.ls_max) {
        if (lane < nf) sm.un[lane] = sm.u[lane] + 0.5 * alpha * sm.pv[lane];
        return optimiser_point(a, sm, EV_SEARCH, f32);
      }
      if (!accepted && lane == 0) sm.status = edm < goal ? FIT_CONVERGED : FIT_LSFAIL;
      gsync<64>();
    } else {
      f = fe;
      go_on = __builtin_isfinite(f);
      gsync<64>();
      if (lane == 0) {
        sm.f = f;
        if (!go_on) sm.status = f == __builtin_inf() ? FIT_DOMAIN : FIT_NONFINITE;
      }
      gsync<64>();
    }
    if (!go_on) {
      if (!(f32 && __builtin_isfinite(f))) return optimiser_end(sm, f, sm.status);
      if (lane < nf) sm.un[lane] = sm.u[lane];
      return optimiser_point(a, sm, EV_FINAL, true);
    }
    differences = fd && nf > 0;  // the gradient, only at accepted points
    if (differences && lane == 0) sm.after = stage;
    if (differences && accepted && lane == 0) sm.fn = fe;
  }
  if (differences) {
    const double uq = sm.un[q], h = kFdStep * fmax(1.0, fabs(uq));
    if (lane == 0) {
      sm.q = q;
      sm.hp = uq + h;
      sm.hm = uq - h;
    }
    if (lane < nf) sm.up[lane] = lane == q ? uq + h : sm.un[lane];
    return optimiser_point(a, sm, EV_FD_PLUS, false);
  }
  // gradient at the new point, in the scaled coordinates.  Lane q < nf holds
  // entry q of every vector and row q of H; the other lanes hold zeros, and
  // rows of H that are never written.  What passes between lanes goes by DPP
  // and readlane, not through LDS in sums of P terms one after the other: one
  // fit of 10,000 bins 77.3 -> 74.6 us, 512 fits of three Gaussians 309 -> 298.
  const bool mine = lane < nf;
  double gq = 0.0;
  if (mine) gq = fd ? sm.gn[lane] : sm.sig[sm.fidx[lane]] * sm.tot[1 + sm.fidx[lane]];
  double h[P];
#pragma unroll
  for (int c = 0; c < P; ++c) h[c] = sm.H[(mine ? lane : 0) * P + c];
  const double un = mine ? sm.un[lane] : 0.0;
  if (accepted) {
    const double sv = mine ? un - sm.u[lane] : 0.0, yv = mine ? gq - sm.g[lane] : 0.0;
    f = fd && nf > 0 ? sm.fn : fe;
    const double sy = lane_sum(sv * yv), yy = lane_sum(yv * yv), ss = lane_sum(sv * sv);
    if (sy > 1e-12 * sqrt(ss) * sqrt(yy)) {
      if (sm.first) {
        const double gam = sy / yy;
#pragma unroll
        for (int c = 0; c < P; ++c) h[c] *= gam;
        gsync<64>();
        if (lane == 0) sm.first = 0;
      }
      const double rho = 1.0 / sy;
      const double Hy = row_times<P>(h, yv);
      const double cc = rho * rho * lane_sum(yv * Hy) + rho;
#pragma unroll
      for (int c = 0; c < P; ++c) {
        const double sc = readlane_d(sv, c), Hc = readlane_d(Hy, c);
        h[c] += -rho * (Hy * sc + sv * Hc) + cc * sv * sc;
        if (mine) sm.H[lane * P + c] = h[c];
      }
    }
  }
  gsync<64>();
  if (mine) {
    sm.u[lane] = un;
    sm.g[lane] = gq;
  }
  if (lane == 0) sm.f = f;
  // direction p = -H g
  if (sm.it < a.max_iter) {
    double pv = mine ? -row_times<P>(h, gq) : 0.0;
    double slope = lane_sum(gq * pv);
    const double edm = -0.5 * slope;
    const double goal = fmax(a.edm_tol, 4.0 * DBL_EPSILON * fabs(f));
    if (f32 && a.polish_edm > 0.0 && edm < a.polish_edm) {
      // switch to FP64 bins for the rest of the fit, at sm.un = sm.u
      if (lane == 0) ++sm.nev;
      if (mine) sm.pv[lane] = pv;
      return optimiser_point(a, sm, EV_POLISH, false);
    }
    if (!a.fixed_iters && edm < goal) {
      if (lane == 0) sm.status = FIT_CONVERGED;
    } else {
      if (!(slope < 0.0)) {  // H lost positive definiteness: restart from I
        for (int t = lane; t < P * P; t += 64) sm.H[t] = (t / P == t % P) ? 1.0 : 0.0;
        pv = -gq;
        if (lane == 0) sm.first = 1;
        slope = -lane_sum(gq * gq);
      }
      if (lane == 0) {
        sm.edm = edm;
        sm.goal = goal;
        sm.slope = slope;
        sm.alpha = 1.0;
        sm.ls = 0;
      }
      if (mine) {
        sm.pv[lane] = pv;
        sm.un[lane] = un + pv;
      }
      return optimiser_point(a, sm, EV_SEARCH, f32);
    }
    gsync<64>();
  }
  if (!f32) return optimiser_end(sm, f, sm.status);
  optimiser_point(a, sm, EV_FINAL, true);  // the NLL at sm.un = sm.u once more with FP64 bins
}

template <int NG, int BKG, int OBJ, int BLK>
__device__ __forceinline__ void fit_one(const FitArgs& a, FitShared<NG, BKG, BLK>& sm,
    const double2* lut, uint32_t* cache, int cache_cap, int b) {
  constexpr int P = FitShared<NG, BKG, BLK>::P;
  constexpr int NB = Shape1D<NG, BKG>::NB;
  const int tid = gtid<BLK>();
  const int64_t off = a.offsets[b];
  const int64_t nb = a.offsets[b + 1] - off;
  const double lo = a.ranges[2 * b], hi = a.ranges[2 * b + 1];
  if (!(nb >= 1) || !(hi > lo) || !__builtin_isfinite(lo) || !__builtin_isfinite(hi)) {
    if (tid < P) a.theta_out[static_cast<int64_t>(b) * P + tid] = a.theta0[static_cast<int64_t>(b) * P + tid];
    if (tid == 0) {
      a.nll_out[b] = __builtin_nan("");
      a.status[b] = FIT_BADHIST;
      a.iters[b] = 0;
      a.nevals[b] = 0;
    }
    gsync<BLK>();
    return;
  }
  const double hx = (hi - lo) / static_cast<double>(nb);
  const double x0 = lo + 0.5 * hx;
  const int S = run_groups<NG>(nb, BLK);
  CountsSrc src{nullptr, a.counts, a.dtype, off};
  if (a.dtype == DT_U32 && nb <= cache_cap) {  // keep the counts in LDS for all evaluations
    const uint32_t* g = static_cast<const uint32_t*>(a.counts) + off;
    for (int64_t i = tid; i < nb; i += BLK) cache[i] = g[i];
    src.lds = cache;
  }

  if (tid < P) sm.th0[tid] = sm.th[tid] = a.theta0[static_cast<int64_t>(b) * P + tid];
  gsync<BLK>();
  if (tid == 0) {
    const double rx = hi - lo;
    int k = 0;
    for (int g = 0; g < NG; ++g, k += 3) {
      sm.sig[k] = fmax(fabs(sm.th0[k]), 1.0);
      sm.sig[k + 1] = rx / 100.0;
      sm.sig[k + 2] = fabs(sm.th0[k + 2]) > 0.0 ? fabs(sm.th0[k + 2]) : rx / 100.0;
    }
    for (int j = 0; j < NB; ++j) sm.sig[k + j] = fmax(fabs(sm.th0[k + j]), 1.0);
    int nf = 0;
    for (int q = 0; q < P; ++q)
      if (a.free_mask == 0u || ((a.free_mask >> q) & 1u)) sm.fidx[nf++] = q;
    sm.nf = nf;
  }
  if (tid < P) sm.u[tid] = sm.un[tid] = 0.0;
  gsync<BLK>();
  const bool lead = tid < 64;
  if (a.hessian_init == 1 && sm.nf > 0) fisher_pass<NG, BKG, OBJ, 0, BLK>(a, sm, src, nb, x0, hx);
  if (lead) optimiser_begin<NG, BKG, OBJ, BLK>(a, sm);
  // The group's first wave runs the optimiser, alone and without group
  // barriers; the others only evaluate, at the point in sm.th.  Every
  // evaluation of a fit passes through this one place, so each sweep is built
  // once per group size.
  for (;;) {
    gsync<BLK>();
    const int cmd = sm.cmd;
    if (cmd == CMD_DONE) break;
    if (cmd == CMD_VALUE)
      wg_eval<NG, BKG, OBJ, false, false, BLK>(a, sm, lut, src, nb, x0, hx, S);
    else if (cmd == CMD_F32)
      wg_eval<NG, BKG, OBJ, true, true, BLK>(a, sm, lut, src, nb, x0, hx, S);
    else
      wg_eval<NG, BKG, OBJ, false, true, BLK>(a, sm, lut, src, nb, x0, hx, S);
    if (lead) optimiser_step<NG, BKG, OBJ, BLK>(a, sm);
  }
  if (!lead) return;
  // final parameters, canonicalised
  if (tid == 0) {
    for (int q = 0; q < sm.nf; ++q) {
      const int k = sm.fidx[q];
      sm.th[k] = fma(sm.sig[k], sm.u[q], sm.th0[k]);
    }
    for (int g = 0; g < NG; ++g) sm.th[3 * g + 2] = fabs(sm.th[3 * g + 2]);
    for (int p = 1; p < NG; ++p)
      for (int q = p; q > 0 && sm.th[3 * q + 1] < sm.th[3 * (q - 1) + 1]; --q)
        for (int r = 0; r < 3; ++r) {
          const double t = sm.th[3 * q + r];
          sm.th[3 * q + r] = sm.th[3 * (q - 1) + r];
          sm.th[3 * (q - 1) + r] = t;
        }
    a.nll_out[b] = sm.nll;
    a.status[b] = sm.status;
    a.iters[b] = sm.it;
    a.nevals[b] = sm.nev;
  }
  gsync<64>();
  if (tid < P) a.theta_out[static_cast<int64_t>(b) * P + tid] = sm.th[tid];
  gsync<64>();
}

// Bytes of dynamic LDS one wave takes in wave mode: its fit state, then an
// LDS copy of up to wave_bins u32 counts, each rounded up to 16 bytes so
// that every slot's counts start 16-byte aligned.
template <int NG, int BKG>
constexpr size_t wave_slot_bytes(int wave_bins) {
  return ((sizeof(FitShared<NG, BKG, 64>) + 15) / 16) * 16 +
         ((4 * static_cast<size_t>(wave_bins) + 15) / 16) * 16;
}

template <int NG, int BKG, int OBJ, int BLK>
__global__ __launch_bounds__(BLK, 2) void k_fit(FitArgs a) {
  __shared__ FitShared<NG, BKG, BLK> sm;
  __shared__ double2 lut[OBJ == OBJ_POISSON ? kLogLut : 1];
  // the workgroup's count cache, or the waves' slots
  extern __shared__ __attribute__((aligned(16))) uint32_t cache[];
  const int tid = threadIdx.x;
  // the log table, by the waves other than the first, which meanwhile starts
  // on the first histogram; fit_one's barriers come before its first use
  if constexpr (OBJ == OBJ_POISSON) {
    if (tid >= 64)
      for (int j = tid - 64; j < kLogLut; j += BLK - 64) lut[j] = a.log_lut[j];
  }
  // The first gridDim.x places of the queue, the longest histograms, belong to
  // the workgroups by index, which spreads them over the CUs (600 histograms of
  // 256..20,000 bins 107 us; with every place from the counter, two of the
  // longest end up on one CU: 146); all workgroups are resident, see launch_fit.
  // The counter hands out the rest.  With no more histograms than workgroups
  // there is no rest, and the queue is not touched (nor re-armed).
  const bool queue = static_cast<int>(gridDim.x) < a.B;
  auto take = [&]() { return queue ? static_cast<int>(gridDim.x + atomicAdd(&a.counters[0], 1u)) : a.B; };
  // wave mode: the order puts every histogram of at most wave_bins bins after
  // all larger ones, so the first of them is followed by such only
  const bool waves = a.wave_bins > 0 && a.sorted;
  int h = blockIdx.x;
  while (h < a.B) {
    const int b = a.sorted ? a.order[h] : h;
    if (waves && a.offsets[b + 1] - a.offsets[b] <= a.wave_bins) break;
    fit_one<NG, BKG, OBJ, BLK>(a, sm, lut, cache, a.cache_bins, b);
    if (tid == 0) sm.h = take();
    __syncthreads();
    h = sm.h;
    __syncthreads();
  }
  if (waves && h < a.B) {
    __syncthreads();  // the log table, where no histogram came before
    // from here on every wave fits its own histograms: wave 0 the one just
    // taken, the others and every later one from the queue
    const int w = tid >> 6;
    char* slot = reinterpret_cast<char*>(cache) + w * wave_slot_bytes<NG, BKG>(a.wave_bins);
    auto& sw = *reinterpret_cast<FitShared<NG, BKG, 64>*>(slot);
    uint32_t* wc = reinterpret_cast<uint32_t*>(slot + wave_slot_bytes<NG, BKG>(0));
    auto take_wave = [&]() {
      int t = 0;
      if ((tid & 63) == 0) t = take();
      return __shfl(t, 0);
    };
    int hw = w == 0 ? h : take_wave();
    while (hw < a.B) {
      fit_one<NG, BKG, OBJ, 64>(a, sw, lut, wc, a.wave_bins, a.order[hw]);
      hw = take_wave();
    }
  }
  if (!queue) return;
  __syncthreads();  // every wave is past the queue before the workgroup leaves
  // the last workgroup to leave re-arms the queue for the next launch
  if (tid == 0) {
    __threadfence();
    const unsigned d = atomicAdd(&a.counters[1], 1u);
    if (d == gridDim.x - 1) {
      atomicExch(&a.counters[0], 0u);
      atomicExch(&a.counters[1], 0u);
    }
  }
}

// grid > 0 launches; 0, -1 and -2 ask, through *answer, for the largest dynamic
// LDS cache (u32 bins) that still fits, for the largest wave_bins whose
// per-wave slots fit, and for the workgroups of a.cache_bins and a.wave_bins
// that are resident on a CU at once.
enum : int { FIT_ASK_CACHE = 0, FIT_ASK_WAVES = -1, FIT_ASK_RESIDENT = -2 };

template <int NG, int BKG, int OBJ, int BLK>
hipError_t launch_fit_kernel(const FitArgs& a, int grid, hipStream_t s, int* answer) {
  size_t dyn = sizeof(uint32_t) * static_cast<size_t>(a.cache_bins);
  if (a.wave_bins > 0) {
    const size_t w = (BLK / 64) * wave_slot_bytes<NG, BKG>(a.wave_bins);
    dyn = w > dyn ? w : dyn;
  }
  if (grid == FIT_ASK_RESIDENT)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(answer, k_fit<NG, BKG, OBJ, BLK>, BLK, dyn);
  if (grid <= 0) {
    hipFuncAttributes attr;
    hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(k_fit<NG, BKG, OBJ, BLK>));
    if (e != hipSuccess) return e;
    int dev = 0, lds = 0;
    e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e != hipSuccess) return e;
    const long free_bytes = static_cast<long>(lds) - static_cast<long>(attr.sharedSizeBytes);
    if (grid == FIT_ASK_CACHE) {
      *answer = static_cast<int>(free_bytes / 4);
    } else {
      const long per_wave = free_bytes / (BLK / 64) - static_cast<long>(wave_slot_bytes<NG, BKG>(0));
      *answer = per_wave > 0 ? static_cast<int>(per_wave / 16) * 4 : 0;
    }
    return hipSuccess;
  }
  hipLaunchKernelGGL((k_fit<NG, BKG, OBJ, BLK>), dim3(grid), dim3(BLK), dyn, s, a);
  return hipGetLastError();
}

using FitLaunchFn = hipError_t (*)(const FitArgs&, int, hipStream_t, int*);

// Workgroup sizes the fitter is built for: 256 threads (one wave per SIMD)
// or 512 (two), the second for batches whose longest fits set the time.
template <int NG, int BKG, int OBJ>
FitLaunchFn pick_fit_blk(int blk) {
  if (blk == 256) return &launch_fit_kernel<NG, BKG, OBJ, 256>;
  if (blk == 512) return &launch_fit_kernel<NG, BKG, OBJ, 512>;
  return nullptr;
}

template <int NG, int BKG>
FitLaunchFn pick_fit_obj(int obj, int blk) {
  switch (obj) {
    case OBJ_NEYMAN:
      return pick_fit_blk<NG, BKG, OBJ_NEYMAN>(blk);
    case OBJ_PEARSON:
      return pick_fit_blk<NG, BKG, OBJ_PEARSON>(blk);
    case OBJ_POISSON:
      return pick_fit_blk<NG, BKG, OBJ_POISSON>(blk);
    default:
      return nullptr;
  }
}

template <int NG>
FitLaunchFn pick_fit_ng(int bkg, int obj, int blk) {
  switch (bkg) {
    case BKG_NONE:
      if constexpr (NG == 0) return nullptr;
      else return pick_fit_obj<NG, BKG_NONE>(obj, blk);
    case 0:
      return pick_fit_obj<NG, 0>(obj, blk);
    case 1:
      return pick_fit_obj<NG, 1>(obj, blk);
    case 2:
      return pick_fit_obj<NG, 2>(obj, blk);
    case 3:
      return pick_fit_obj<NG, 3>(obj, blk);
    case BKG_EXP:
      return pick_fit_obj<NG, BKG_EXP>(obj, blk);
    default:
      return nullptr;
  }
}

FitLaunchFn pick_fit_ng0(int bkg, int obj, int blk);
FitLaunchFn pick_fit_ng1(int bkg, int obj, int blk);
FitLaunchFn pick_fit_ng2(int bkg, int obj, int blk);
FitLaunchFn pick_fit_ng3(int bkg, int obj, int blk);
FitLaunchFn pick_fit_ng4(int bkg, int obj, int blk);

}  // namespace hf
