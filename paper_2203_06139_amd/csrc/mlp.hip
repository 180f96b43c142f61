// mlp.hip -- learned initialiser: rebinning, default starts, target maps and
// column statistics (the network's kernels are in mlp_net.hip).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.hpp"
#include "mlp.hpp"

namespace hf {

// ---------------------------------------------------------------------------
// Histogram -> network input, default starts, target maps, column statistics
// ---------------------------------------------------------------------------
__device__ __forceinline__ double count_any(const void* base, int dtype, int64_t i) {
  if (dtype == DT_U32) return static_cast<const uint32_t*>(base)[i];
  if (dtype == DT_F32) return static_cast<const float*>(base)[i];
  return static_cast<const double*>(base)[i];
}

// Fine bin i goes to coarse bin floor((2i+1) 256 / (2 nb)); the fine bins of
// coarse bin j are i in [lo(j), lo(j+1)) with lo(j) the count of i whose
// (2i+1) 256 < 2 j nb, i.e. lo(j) = ceil((2 j nb - 256) / 512) clamped.
// I: 64 bits, or 32 where nb allows (kShort).
template <class I>
__device__ __forceinline__ I run_start(int j, I nb) {
  if (j == kMlpIn) return nb;
  const I num = 2 * static_cast<I>(j) * nb - kMlpIn;
  if (num <= 0) return 0;
  const I q = (num + 2 * kMlpIn - 1) / (2 * kMlpIn);
  return q < nb ? q : nb;
}
constexpr int64_t kShort = 1 << 21;  // 2 j nb + 511 stays below 2^31

// Rebinning: one block per histogram; from six counts per coarse bin on S =
// 2^slog lanes each, S the largest power of two not above the run length nb / 256
// (at most 16, a DPP row): lane s takes the run's bins s, s + S, ..., so a wave reads segments of
// up to 64 bytes, and the S partial sums meet in DPP moves.  U coarse bins are
// summed side by side over R segments each, which keeps U R loads per lane in
// flight; positions past a run's end are clamped into the histogram and
// dropped.  Sums of integer-valued counts are exact in FP64 in any order;
// others are added in a fixed order.
// Bound: HBM, one read of the counts, and for the mid sizes the instructions
// around a load (with 64-bit positions 46.6 us for 4096 histograms of 10,000
// bins, with 32-bit ones and S known to the compiler 35.6).  4096 histograms of
// 256..65536 bins (193 MB of u32 counts): 509 us (0.38 TB/s) with one thread
// walking each run through memory, 59.5 us with (U, R) = (8, 1) and 64-bit
// positions, 46.2 us (4.1 TB/s) now.  (U, R) in us for that batch, for 4096 of
// 10,000 bins and for 1024 of 60,000 to 65,536, where fewer streams read
// faster: (8, 1) 50.0, 35.7, 53.8; (4, 2) 51.5, 39.6, 44.3; (2, 4) 54.4, 41.6,
// 40.6; (8, 2) 46.8, 37.5, 54.0; (4, 4) 46.2, 36.3, 46.7; (2, 8) 55.2, 57.2,
// 40.0.  With up to 64 lanes per run and shuffles the reduction outweighs the
// loads (101 us for the first), with up to 8 lanes 71.
template <int slog, int U, int R, class I, class T>
__device__ __forceinline__ void rebin_runs(const T* __restrict__ c, I nb, double* sum) {
  static_assert(slog >= 2, "quads at least");
  constexpr int S = 1 << slog;
  const int s = threadIdx.x & (S - 1), group = threadIdx.x >> slog, groups = kMlpIn >> slog;
  const I longest = (nb + kMlpIn - 1) / kMlpIn;  // no run is longer
  for (int it = 0; it < S; it += U) {
    I i0[U], len[U];
    double acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = group + (it + u) * groups;
      i0[u] = run_start<I>(j, nb);
      len[u] = run_start<I>(j + 1, nb) - i0[u];
      acc[u] = 0.0;
    }
    for (I k0 = s; k0 - s < longest; k0 += R * S) {  // same trips in every lane
      T v[R][U];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const I i = i0[u] + k0 + r * S;
          v[r][u] = c[i < nb ? i : nb - 1];
        }
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < U; ++u)
          acc[u] += static_cast<double>(k0 + r * S < len[u] ? v[r][u] : static_cast<T>(0));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[u] += dpp_row<0xb1>(acc[u]);                 // quad_perm [1,0,3,2]
      acc[u] += dpp_row<0x4e>(acc[u]);                 // quad_perm [2,3,0,1]
      if (slog > 2) acc[u] += dpp_row<0x141>(acc[u]);  // row_half_mirror: the other quad of 8
      if (slog > 3) acc[u] += dpp_row<0x140>(acc[u]);  // row_mirror: the other 8 of 16
    }
    if (s == 0) {
#pragma unroll
      for (int u = 0; u < U; ++u) sum[group + (it + u) * groups] = acc[u];
    }
  }
}

// Sum of the n counts from i0 by one thread, R in flight.
template <int R, class I, class T>
__device__ __forceinline__ double own_run(const T* __restrict__ c, I nb, I i0, I n) {
  const I longest = (nb + kMlpIn - 1) / kMlpIn;
  double s = 0.0;
  for (I k0 = 0; k0 < longest; k0 += R) {
    T v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = c[i0 + k0 + r < nb ? i0 + k0 + r : nb - 1];
#pragma unroll
    for (int r = 0; r < R; ++r) s += static_cast<double>(k0 + r < n ? v[r] : static_cast<T>(0));
  }
  return s;
}

// Mean of coarse bin threadIdx.x's counts, 0 where it has none.  Runs of up to
// six counts are left to the bin's own thread, without LDS and a barrier: 4096
// histograms of 100, 700, 1020, 1500 and 2040 bins 9.0, 9.7, 10.4, 11.6, 19.7 us,
// with lanes per run 10.3, 12.0, 12.3, 14.0, 14.3 (a thread walking the run one
// count after the other: 9.3, 10.4, 12.0, 13.1, 22.6).
template <class I, class T>
__device__ __forceinline__ double coarse_mean(const T* __restrict__ c, I nb, double* sum) {
  const int j = threadIdx.x;
  const I i0 = run_start<I>(j, nb), n = run_start<I>(j + 1, nb) - i0;
  double s;
  if (nb < 512) {
    s = own_run<2, I>(c, nb, i0, n);
  } else if (nb < 1536) {
    s = own_run<4, I>(c, nb, i0, n);
  } else {
    if (nb >= 4096)
      rebin_runs<4, 4, 4, I>(c, nb, sum);
    else if (nb >= 2048)
      rebin_runs<3, 8, 1, I>(c, nb, sum);
    else
      rebin_runs<2, 4, 1, I>(c, nb, sum);
    __syncthreads();
    s = sum[j];
  }
  return n > 0 ? s / static_cast<double>(n) : 0.0;
}

template <class T>
__global__ __launch_bounds__(kMlpIn) void k_rebin_lognorm(const T* __restrict__ counts,
                                                          const int64_t* __restrict__ offsets,
                                                          float in_mean, float in_std,
                                                          float* __restrict__ out) {
  __shared__ double sum[kMlpIn];
  const int b = blockIdx.x;
  const int64_t off = offsets[b];
  const int64_t nb = offsets[b + 1] - off;
  double mean = 0.0;  // of an empty histogram (uniform over the block)
  if (nb >= kShort)
    mean = coarse_mean<int64_t>(counts + off, nb, sum);
  else if (nb >= 1)
    mean = coarse_mean<int>(counts + off, static_cast<int>(nb), sum);
  out[static_cast<int64_t>(b) * kMlpIn + threadIdx.x] =
      static_cast<float>((log1p(mean) - in_mean) / in_std);
}

hipError_t rebin_lognorm(int B, const void* counts, int dtype, const int64_t* offsets, float mean,
                         float std, float* out, hipStream_t s) {
  if (dtype == DT_U32)
    hipLaunchKernelGGL(k_rebin_lognorm<uint32_t>, dim3(B), dim3(kMlpIn), 0, s,
                       static_cast<const uint32_t*>(counts), offsets, mean, std, out);
  else if (dtype == DT_F32)
    hipLaunchKernelGGL(k_rebin_lognorm<float>, dim3(B), dim3(kMlpIn), 0, s,
                       static_cast<const float*>(counts), offsets, mean, std, out);
  else
    hipLaunchKernelGGL(k_rebin_lognorm<double>, dim3(B), dim3(kMlpIn), 0, s,
                       static_cast<const double*>(counts), offsets, mean, std, out);
  return hipGetLastError();
}

// Default starting point for Gauss + exp(b0 + b1 t); one block per histogram.
//   background: mean counts of the first and last ne = max(nb/25, 1) bins
//     (at least 1), an exponential through the two edge-block centres (the
//     model's own background form; a straight line would leave a false
//     excess at the steep edge of a falling or rising background);
//   peak: the window position i in [W, nb - W), W = max(nb/256, 1), with the
//     largest integer excess e(i) = rint(S(i) - (2W+1) bg(i)), S(i) the sum
//     of counts over [i - W, i + W] (first such i on ties);
//   width: walking out from the peak while 2 e >= e_max, the half-maximum
//     bounds give the FWHM.
// The window positions are split among the block's waves in
// contiguous ranges; a wave walks its range 64 positions per step, lane l
// at position s + l, with coalesced loads: the window sum at position i is
// the sum at the range's first position plus the lane prefix sum of the
// differences c[i + W] - c[i - W - 1] (S(i) - S(i - 1)).  Sums of
// integer-valued counts are exact in FP64 in any order, so every window sum
// and decision matches a direct evaluation; the excess is evaluated without
// FMA contraction (separate products and sums).  The walk for the width
// becomes a search for the nearest positions left and right of the peak
// with 2 e < e_max.
struct Excess {
  double lb0, dlb, c0, cden, wlen;
  __device__ __forceinline__ int64_t operator()(double S, int64_t i) const {
#pragma clang fp contract(off)
    const double bg = exp(lb0 + dlb * ((static_cast<double>(i) + 0.5 - c0) / cden));
    return static_cast<int64_t>(__builtin_rint(S - wlen * bg));
  }
};

// Calls fn(S, i) for every window position i of [q0, q1) (one wave, lane l
// taking positions q0 + l, q0 + 64 + l, ...), S the window sum over
// [i - W, i + W].
template <class Fn>
__device__ __forceinline__ void window_walk(const void* counts, int dtype, int64_t off, int64_t q0,
                                            int64_t q1, int64_t W, Fn fn) {
  if (q0 >= q1) return;
  const int lane = static_cast<int>(threadIdx.x & 63u);
  double s0 = 0.0;
  for (int64_t q = q0 - W + lane; q <= q0 + W; q += 64) s0 += count_any(counts, dtype, off + q);
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) s0 += __shfl_xor(s0, k);
  double carry = s0;  // S(q0), then S of the previous step's last position
  for (int64_t base = q0; base < q1; base += 64) {
    const int64_t i = base + lane;
    double d = 0.0;
    if (i > q0 && i < q1)
      d = count_any(counts, dtype, off + i + W) - count_any(counts, dtype, off + i - W - 1);
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
      const double u = __shfl_up(d, k);
      if (lane >= k) d += u;
    }
    const double S = carry + d;
    if (i < q1) fn(S, i);
    carry = __shfl(S, 63);
  }
}

// The same sums for u32 counts, which are integers: exact in any order, so the
// prefix goes by DPP, and the next step's counts are requested ahead.  fn(S, i,
// in) is called by the whole wave, whose walk ends where it returns true.
__device__ __forceinline__ double wave_prefix(double d) {
  const int row = static_cast<int>(threadIdx.x & 63u) >> 4;
  d += dpp_row<0x111>(d);  // row_shr:1, 2, 4, 8
  d += dpp_row<0x112>(d);
  d += dpp_row<0x114>(d);
  d += dpp_row<0x118>(d);
  const double a = readlane_d(d, 15), ab = a + readlane_d(d, 31), abc = ab + readlane_d(d, 47);
  return d + (row == 0 ? 0.0 : row == 1 ? a : row == 2 ? ab : abc);
}

template <class Fn>
__device__ __forceinline__ void window_walk_u32(const uint32_t* __restrict__ c, int64_t q0, int64_t q1,
                                                int64_t W, Fn fn) {
  if (q0 >= q1) return;
  const int lane = static_cast<int>(threadIdx.x & 63u);
  double s0 = 0.0;
#pragma unroll 4
  for (int64_t q = q0 - W + lane; q <= q0 + W; q += 64) s0 += c[q];
  double carry = wave_sum(s0);  // S(q0), then S of the previous step's last position
  auto step = [&](int64_t i) {  // S(i) - S(i - 1)
    return i > q0 && i < q1 ? static_cast<double>(c[i + W]) - static_cast<double>(c[i - W - 1]) : 0.0;
  };
  double next = step(q0 + lane);
  for (int64_t base = q0; base < q1; base += 64) {
    const int64_t i = base + lane;
    const double S = carry + wave_prefix(next);
    next = step(i + 64);
    if (fn(S, i, i < q1)) return;
    carry = readlane_d(S, 63);
  }
}

// T threads per histogram.  U32 (u32 counts): 512, which the registers of its
// estimates allow two blocks per CU; otherwise 1024, with the walk above.
// 4096 histograms of 256..65536 bins: 2.86 ms when each thread walked its own
// segment of positions with scattered loads, 0.88 ms with 16 waves and every
// excess (an exp and a division) rounded as the direct evaluation does, twice;
// 0.47 ms with the excess only where an estimate leaves it a chance, and the
// width searched outwards from the peak.  In us, walked twice and now: 4096 of
// 64..512 bins 182 and 71, 4096 of 10,000 516 and 256, 64 of 65,536 153 and 105;
// one of 1e6 with a peak of 2% of the range 2144 and 1236, of 10% 2142 and
// 1706, without a peak 2105 and 2135 (the search then covers all of it).  (With
// 1 to 6% more time per position, before the loops' constants were
// materialised in them:) with 1024 threads one block fits a CU (670,
// 458, 66.7), with spills two (884, 581, 79.2); 256 threads take 476, 231 and
// 22.2, but 251 us instead of 160 for 64 histograms of 65,536.
template <int T, bool U32>
__global__ __launch_bounds__(T, 4) void k_default_starts(const void* counts, int dtype,
                                                               const int64_t* __restrict__ offsets,
                                                               const double* __restrict__ ranges,
                                                               double t_shift, double t_scale,
                                                               double* __restrict__ theta0) {
  constexpr int kWavesDs = T / 64;
  __shared__ double red_d[2][kWavesDs];
  __shared__ int64_t red_e[kWavesDs];
  __shared__ int64_t red_i[kWavesDs];
  __shared__ int64_t red_j[kWavesDs];
  const int b = blockIdx.x;
  const int t = threadIdx.x;
  const int lane = t & 63, wv = t >> 6;
  const int64_t off = offsets[b];
  const int64_t nb = offsets[b + 1] - off;
  if (nb < 1) {  // empty histogram: no start (uniform over the block)
    if (t < 5) theta0[static_cast<int64_t>(b) * 5 + t] = __builtin_nan("");
    return;
  }
  const double lo = ranges[2 * b], hi = ranges[2 * b + 1];
  const double h = (hi - lo) / static_cast<double>(nb);
  const int64_t ne = nb / 25 > 0 ? nb / 25 : 1;  // 4% of the bins at each edge
  // edge sums (integer-valued: exact in any order)
  double sl = 0.0, sr = 0.0;
  for (int64_t i = t; i < ne; i += T) {
    sl += count_any(counts, dtype, off + i);
    sr += count_any(counts, dtype, off + nb - ne + i);
  }
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) {
    sl += __shfl_xor(sl, k);
    sr += __shfl_xor(sr, k);
  }
  if (lane == 0) {
    red_d[0][wv] = sl;
    red_d[1][wv] = sr;
  }
  __syncthreads();
  double esl = 0.0, esr = 0.0;
#pragma unroll
  for (int w = 0; w < kWavesDs; ++w) {
    esl += red_d[0][w];
    esr += red_d[1][w];
  }
  const double bk0 = fmax(esl / static_cast<double>(ne), 1.0);
  const double bk1 = fmax(esr / static_cast<double>(ne), 1.0);
  const double c0 = 0.5 * static_cast<double>(ne);
  const double c1 = static_cast<double>(nb) - 0.5 * static_cast<double>(ne);
  const int64_t W = nb / 256 > 1 ? nb / 256 : 1;
  const double lb0 = log(bk0);
  const Excess ex{lb0, log(bk1) - lb0, c0, c1 - c0, static_cast<double>(2 * W + 1)};
  // this wave's range [q0, q1) of the window positions [W, nb - W)
  const int64_t nv = nb - 2 * W > 0 ? nb - 2 * W : 0;
  const int64_t Lw = (nv + kWavesDs - 1) / kWavesDs;
  const int64_t q0 = W + wv * Lw;
  const int64_t q1 = (W + (wv + 1) * Lw < nb - W) ? W + (wv + 1) * Lw : nb - W;
  // pass 1: largest excess, first position (per lane, positions increase)
  int64_t be = INT64_MIN, bi = 0;
  // window sums of u32 counts stay below 2^53, so they are exact
  const bool whole = U32 && W < (1 << 20);
  const uint32_t* cu = static_cast<const uint32_t*>(counts) + off;
  const double rc = 1.0 / ex.cden;
  auto background = [&](int64_t i) {  // of the window, to 1e-9 and far better
    return ex.wlen * exp_fast(fma(ex.dlb, (static_cast<double>(i) + 0.5 - ex.c0) * rc, ex.lb0));
  };
  if (whole) {
    // The excess as it has to round is evaluated only where a close estimate
    // (1e-9 of the background is far above its error) leaves it a chance of
    // exceeding the wave's largest so far: a dozen steps of a wave's range.
    window_walk_u32(cu, q0, q1, W, [&](double S, int64_t i, bool in) {
      const double bg = background(i);
      const bool chance = in && !(fma(1e-9, bg, S - bg) < static_cast<double>(be) + 0.25);
      if (__any(chance)) {
        // an excess is below 2^53 in size: its double is the integer
        const double e = chance ? static_cast<double>(ex(S, i)) : -1e19;
        double m = fmax(e, dpp_row<0x128>(e));
        m = fmax(m, dpp_row<0x124>(m));
        m = fmax(m, dpp_row<0x4e>(m));
        m = fmax(m, dpp_row<0xb1>(m));
        m = fmax(fmax(readlane_d(m, 0), readlane_d(m, 16)), fmax(readlane_d(m, 32), readlane_d(m, 48)));
        if (m > static_cast<double>(be)) {
          be = static_cast<int64_t>(m);
          bi = i - lane + __builtin_ctzll(__ballot(e == m));
        }
      }
      return false;
    });
  } else {
    window_walk(counts, dtype, off, q0, q1, W, [&](double S, int64_t i) {
      const int64_t e = ex(S, i);
      if (e > be) {
        be = e;
        bi = i;
      }
    });
  }
  // the largest excess, the first position among equals: over the lanes,
  // then over the waves
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) {
    const int64_t oe = __shfl_xor(be, k), oi = __shfl_xor(bi, k);
    if (oe > be || (oe == be && oi < bi)) {
      be = oe;
      bi = oi;
    }
  }
  if (lane == 0) {
    red_e[wv] = be;
    red_i[wv] = bi;
  }
  __syncthreads();
  int64_t emax = INT64_MIN, imax = nb / 2;
#pragma unroll
  for (int w = 0; w < kWavesDs; ++w)
    if (red_e[w] > emax || (red_e[w] == emax && red_i[w] < imax)) {
      emax = red_e[w];
      imax = red_i[w];
    }
  if (emax == INT64_MIN) {  // histogram shorter than one window
    emax = 0;
    imax = nb / 2;
  }
  __syncthreads();
  // pass 2: nearest positions left / right of the peak with 2 e < emax
  int64_t pl = INT64_MIN, pr = INT64_MAX;
  if (whole) {
    // Outwards from the peak until both are found: half of the waves on each
    // side, all of them on the side that is left.  A wave takes a stretch of L
    // positions per round, a window's length (four where one side is left, which
    // is then long), so that the window sum it starts from costs no more than
    // the walk, and a search of n positions reads less than 3 n counts; the
    // excess is evaluated as in pass 1, where an estimate leaves it a chance to
    // be below half of the peak's.
    const int64_t L0 = (2 * W + 64) / 64 * 64;
    const double below = static_cast<double>((emax - 1) >> 1) + 0.75;
    int64_t dl = 0, dr = 0;  // positions searched on each side
    bool more_l = imax > W, more_r = imax + 1 < nb - W;
    while (more_l || more_r) {
      const int64_t L = more_l && more_r ? L0 : 4 * L0;
      const int nr = !more_r ? 0 : (more_l ? kWavesDs / 2 : kWavesDs);
      const bool right = wv < nr;
      const int64_t w0 = right ? imax + 1 + dr + L * wv : imax - dl - L * (wv - nr + 1);
      int64_t fl = INT64_MIN, fr = INT64_MAX;
      window_walk_u32(cu, w0 > W ? w0 : W, w0 + L < nb - W ? w0 + L : nb - W, W,
                      [&](double S, int64_t i, bool in) {
                        bool chance = in;
                        if (dl + dr > 0) {  // in the first round most have one
                          const double bg = background(i);
                          chance = in && fma(-1e-9, bg, S - bg) < below;
                          if (!__any(chance)) return false;
                        }
                        const uint64_t hit = __ballot(chance && 2 * ex(S, i) < emax);
                        if (!hit) return false;
                        if (right)
                          fr = i - lane + __builtin_ctzll(hit);  // the first
                        else
                          fl = i - lane + 63 - __builtin_clzll(hit);  // the last so far
                        return right;
                      });
      if (lane == 0) {
        red_e[wv] = fl;
        red_j[wv] = fr;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kWavesDs; ++w) {
        pl = red_e[w] > pl ? red_e[w] : pl;
        pr = red_j[w] < pr ? red_j[w] : pr;
      }
      dr += nr * L;
      dl += (kWavesDs - nr) * L;
      more_l = more_l && pl == INT64_MIN && imax - dl > W;
      more_r = more_r && pr == INT64_MAX && imax + 1 + dr < nb - W;
      __syncthreads();
    }
  } else {
    window_walk(counts, dtype, off, q0, q1, W, [&](double S, int64_t i) {
      if (i != imax && 2 * ex(S, i) < emax) {
        if (i < imax) pl = i > pl ? i : pl;  // the largest below the peak
        else pr = i < pr ? i : pr;           // the smallest above it
      }
    });
  }
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) {
    const int64_t ol = __shfl_xor(pl, k), orr = __shfl_xor(pr, k);
    pl = ol > pl ? ol : pl;
    pr = orr < pr ? orr : pr;
  }
  if (lane == 0) {
    red_e[wv] = pl;
    red_j[wv] = pr;
  }
  __syncthreads();
  if (t == 0) {
    int64_t l = INT64_MIN, r = INT64_MAX;
    for (int q = 0; q < kWavesDs; ++q) {
      l = red_e[q] > l ? red_e[q] : l;
      r = red_j[q] < r ? red_j[q] : r;
    }
    // the walk stops just inside the first failing position, or at the edge
    // of the window range; it never moves when that range is empty
    const int64_t left = l == INT64_MIN ? W : (l + 1 > W ? l + 1 : W);
    const int64_t right = r == INT64_MAX ? nb - W - 1 : (r - 1 < nb - W - 1 ? r - 1 : nb - W - 1);
    const int64_t b0i = left < imax ? left : imax;
    const int64_t b1i = right > imax ? right : imax;
    const double range = hi - lo;
    const double fwhm = static_cast<double>(b1i - b0i + 1) * h;
    const double s = fmin(fmax(fwhm / 2.3548200450309493, 0.005 * range), 0.1 * range);
    const double A = fmax(static_cast<double>(emax) / ex.wlen, 1.0);
    const double m = lo + (static_cast<double>(imax) + 0.5) * h;
    const double t0 = (lo + c0 * h - t_shift) / t_scale;
    const double t1 = (lo + c1 * h - t_shift) / t_scale;
    const double b1 = log(bk1 / bk0) / (t1 - t0);
    const double b0v = log(bk0) - b1 * t0;
    double* th = theta0 + static_cast<int64_t>(b) * 5;
    th[0] = A;
    th[1] = m;
    th[2] = s;
    th[3] = b0v;
    th[4] = b1;
  }
}

hipError_t default_starts(int B, const void* counts, int dtype, const int64_t* offsets,
                          const double* ranges, double t_shift, double t_scale, double* theta0,
                          hipStream_t s) {
  if (dtype == DT_U32)
    hipLaunchKernelGGL((k_default_starts<512, true>), dim3(B), dim3(512), 0, s, counts, dtype, offsets,
                       ranges, t_shift, t_scale, theta0);
  else
    hipLaunchKernelGGL((k_default_starts<1024, false>), dim3(B), dim3(1024), 0, s, counts, dtype,
                       offsets, ranges, t_shift, t_scale, theta0);
  return hipGetLastError();
}

__global__ void k_theta_to_target(int B, const double* __restrict__ th, const float* mean,
                                  const float* std, float* __restrict__ t) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const double* p = th + static_cast<int64_t>(b) * 5;
  const double raw[5] = {p[1], log(fabs(p[2])), log(fabs(p[0])), p[3], p[4]};
  for (int k = 0; k < 5; ++k)
    t[static_cast<int64_t>(b) * 5 + k] = static_cast<float>((raw[k] - mean[k]) / std[k]);
}

__global__ void k_target_to_theta(int B, const float* __restrict__ y, const float* mean,
                                  const float* std, double* __restrict__ th) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  double v[5];
  for (int k = 0; k < 5; ++k)
    v[k] = static_cast<double>(y[static_cast<int64_t>(b) * kMlpOutPad + k]) * std[k] + mean[k];
  double* p = th + static_cast<int64_t>(b) * 5;
  p[0] = exp(v[2]);
  p[1] = v[0];
  p[2] = exp(v[1]);
  p[3] = v[3];
  p[4] = v[4];
}

hipError_t theta_to_target(int B, const double* th, const float* mean, const float* std, float* t,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_theta_to_target, dim3((B + 255) / 256), dim3(256), 0, s, B, th, mean, std, t);
  return hipGetLastError();
}

hipError_t target_to_theta(int B, const float* y, const float* mean, const float* std, double* th,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_target_to_theta, dim3((B + 255) / 256), dim3(256), 0, s, B, y, mean, std, th);
  return hipGetLastError();
}

// One block per column: FP64 sum and sum of squares over rows in a fixed
// (strided, then tree) order.
__global__ __launch_bounds__(256) void k_column_stats(int64_t n, int cols, const float* __restrict__ x,
                                                      float* mean, float* stdv) {
  __shared__ double s1[256], s2[256];
  const int c = blockIdx.x;
  double a = 0.0, q = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) {
    const double v = x[i * cols + c];
    a += v;
    q += v * v;
  }
  s1[threadIdx.x] = a;
  s2[threadIdx.x] = q;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      s1[threadIdx.x] += s1[threadIdx.x + w];
      s2[threadIdx.x] += s2[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double mu = s1[0] / static_cast<double>(n);
    const double var = fmax(s2[0] / static_cast<double>(n) - mu * mu, 0.0);
    mean[c] = static_cast<float>(mu);
    stdv[c] = static_cast<float>(var > 0.0 ? sqrt(var) : 1.0);
  }
}

hipError_t column_stats(int64_t n, int cols, const float* x, float* mean, float* stdv,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_column_stats, dim3(cols), dim3(256), 0, s, n, cols, x, mean, stdv);
  return hipGetLastError();
}

}  // namespace hf
