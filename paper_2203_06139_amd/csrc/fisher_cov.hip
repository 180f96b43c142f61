// fisher_cov.hip -- parameter covariance from Fisher matrices, one wave per
// matrix.
//
// For the free parameters (free_mask bit set, or all when the mask is 0):
//   S = diag(F)^(-1/2),  R = S F S (unit diagonal),
//   R = L L^T (Cholesky; every pivot must exceed 1e-12 and be finite),
//   cov = scale * S inv(L)^T inv(L) S.
// Scaling to unit diagonal first makes the pivot test independent of the
// parameters' units (an amplitude of 1e4 counts next to a width of 0.01).
// The rows and columns of fixed parameters are 0.  A free block that is not
// safely positive definite (or a non-positive diagonal entry) gives NaN in
// the free entries and status 1.
#include "fisher_kernels.hpp"

namespace hf {

constexpr int kCovMaxP = 16;

// Lane r holds row r of R and L over the free parameters, then column r of
// inv(L), in registers, and takes the other lanes' values by readlane; rows
// past the free ones (up to N, a multiple of 4) are the identity's.
// Bound: the latency of one chain (N square roots and twice N divisions that
// follow each other).  One 10 x 10 matrix: 12.0 us with the matrix in LDS and
// a barrier per column and per pivot, 6.1 us now.
template <int N>
__global__ __launch_bounds__(64) void k_fisher_cov(const double* __restrict__ F, int P,
                                                   uint32_t free_mask, double scale,
                                                   double* __restrict__ cov,
                                                   int32_t* __restrict__ status) {
  const int r = threadIdx.x;
  const int64_t b = blockIdx.x;
  const double* Fb = F + b * P * P;
  double* Cb = cov + b * P * P;
  const uint32_t all = (1u << P) - 1u;
  const uint32_t mask = free_mask == 0u ? all : (free_mask & all);
  const int nf = __builtin_popcount(mask);
  // index of the r-th free parameter (this lane's) and of every one
  int kr = 0, kc[N];
  uint32_t left = mask;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    kc[c] = left ? __builtin_ctz(left) : 0;
    left &= left - 1u;
    if (c == r) kr = kc[c];
  }
  const bool mine = r < nf;
  double a[N], x[N];
  const double d = mine ? Fb[kr * P + kr] : 1.0;
#pragma unroll
  for (int c = 0; c < N; ++c) a[c] = mine && c < nf ? Fb[kr * P + kc[c]] : 0.0;
  bool ok = d > 0.0 && __builtin_isfinite(d);
  const double sc = 1.0 / sqrt(d);
#pragma unroll
  for (int c = 0; c < N; ++c)
    a[c] = mine && c < nf ? a[c] * sc * readlane_d(sc, c) : (r == c ? 1.0 : 0.0);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const double p = readlane_d(a[j], j);
    if (!(p > 1e-12) || !__builtin_isfinite(p)) ok = false;  // 1 past the free rows
    const double piv = sqrt(p);
    a[j] = r == j ? piv : a[j] / piv;
#pragma unroll
    for (int c = j + 1; c < N; ++c) a[c] = fma(-a[j], readlane_d(a[j], c), a[c]);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double v = r == i ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < i; ++k) v = fma(-readlane_d(a[k], i), x[k], v);
    x[i] = v / readlane_d(a[i], i);
  }
  ok = __all(ok);
  // rows and columns of fixed parameters
  for (int t = r; t < P * P; t += 64)
    if (!((mask >> (t / P)) & (mask >> (t % P)) & 1u)) Cb[t] = 0.0;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    double v = 0.0;
#pragma unroll
    for (int k = c; k < N; ++k) v = fma(x[k], readlane_d(x[k], c), v);
    v *= scale * sc * readlane_d(sc, c);
    if (mine && c < nf) Cb[kr * P + kc[c]] = ok ? v : __builtin_nan("");
  }
  if (r == 0 && status) status[b] = ok ? 0 : 1;
}

hipError_t fisher_covariance(int B, int P, const double* F, uint32_t free_mask, double scale,
                             double* cov, int32_t* status, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  if (P < 1 || P > kCovMaxP) return hipErrorInvalidValue;
  const uint32_t all = (1u << P) - 1u;
  const int nf = __builtin_popcount(free_mask == 0u ? all : (free_mask & all));
  const auto k = nf <= 4 ? k_fisher_cov<4>
                         : (nf <= 8 ? k_fisher_cov<8> : (nf <= 12 ? k_fisher_cov<12> : k_fisher_cov<16>));
  hipLaunchKernelGGL(k, dim3(B), dim3(64), 0, s, F, P, free_mask, scale, cov, status);
  return hipGetLastError();
}

}  // namespace hf
