// fit.hip -- fitter scratch, the longest-first ordering kernel and the launch
// of the persistent fit kernel.
#include <algorithm>

#include "fit_impl.hpp"

namespace hf {

namespace {

constexpr int kMaxRankB = 1 << 16;

// Order of a batch: histograms of more than `split` bins first, and within
// each part longest first to 1/32 of a size, by a counting sort of one block
// over buckets of 32 per octave (the size's FP32 exponent and top mantissa
// bits).  Within a bucket the order is that of the LDS atomics: every fit's
// result is its own, whatever runs beside or before it.  The wave mode of the
// fit kernel needs the split to be exact, hence the two parts.
// Bound: latency of two passes over the sizes.  It replaced a bitonic sort in
// LDS (4096 histograms: 57 us) and, above 4096, a comparison of every pair
// (16,384: 1.0 ms).
constexpr int kSortThreads = 1024;
constexpr int kSortBuckets = 32 * 64;  // sizes below 2^64
constexpr int kSortPer = 2 * kSortBuckets / kSortThreads;

__device__ __forceinline__ int size_bucket(int64_t size, int64_t split) {
  const float f = size < 1 ? 1.0f : static_cast<float>(size);
  const int up = static_cast<int>((__float_as_uint(f) >> 18) - (127u << 5));  // ascending, >= 0
  return (size <= split ? kSortBuckets : 0) + (kSortBuckets - 1 - up);
}

__global__ __launch_bounds__(kSortThreads) void k_sort_sizes(const int64_t* __restrict__ offsets,
                                                             int B, int64_t split,
                                                             int32_t* __restrict__ order) {
  __shared__ int bucket[2 * kSortBuckets];
  __shared__ int wave_total[kSortThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63;
  for (int i = tid; i < 2 * kSortBuckets; i += kSortThreads) bucket[i] = 0;
  __syncthreads();
  // a wave whose histograms all share a bucket (equal sizes) adds them at once
  auto add = [&](int k, bool in) {
    const uint64_t mask = __ballot(in);
    const int k0 = __builtin_amdgcn_readfirstlane(k);
    if (__ballot(in && k != k0) == 0) {
      int base = 0;
      if (lane == 0) base = atomicAdd(&bucket[k0], __popcll(mask));
      base = __builtin_amdgcn_readfirstlane(base);
      return base + static_cast<int>(__popcll(mask & ((uint64_t(1) << lane) - 1)));
    }
    return in ? atomicAdd(&bucket[k], 1) : 0;
  };
  for (int i0 = 0; i0 < B; i0 += kSortThreads) {
    const int i = min(i0 + tid, B - 1);
    add(size_bucket(offsets[i + 1] - offsets[i], split), i0 + tid < B);
  }
  __syncthreads();
  // exclusive scan of the counts: a thread's own buckets, lanes, waves
  int mine[kSortPer], sum = 0;
#pragma unroll
  for (int q = 0; q < kSortPer; ++q) {
    mine[q] = bucket[tid * kSortPer + q];
    sum += mine[q];
  }
  int up = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(up, d);
    if (lane >= d) up += o;
  }
  if (lane == 63) wave_total[tid >> 6] = up;
  __syncthreads();
  int at = up - sum;
  for (int w = 0; w < (tid >> 6); ++w) at += wave_total[w];
#pragma unroll
  for (int q = 0; q < kSortPer; ++q) {
    bucket[tid * kSortPer + q] = at;
    at += mine[q];
  }
  __syncthreads();
  for (int i0 = 0; i0 < B; i0 += kSortThreads) {
    const int i = min(i0 + tid, B - 1);
    const bool in = i0 + tid < B;
    const int p = add(size_bucket(offsets[i + 1] - offsets[i], split), in);
    if (in) order[p] = i;
  }
}

FitLaunchFn pick_fit(int ng, int bkg, int obj, int blk) {
  switch (ng) {
    case 0:
      return pick_fit_ng0(bkg, obj, blk);
    case 1:
      return pick_fit_ng1(bkg, obj, blk);
    case 2:
      return pick_fit_ng2(bkg, obj, blk);
    case 3:
      return pick_fit_ng3(bkg, obj, blk);
    case 4:
      return pick_fit_ng4(bkg, obj, blk);
    default:
      return nullptr;
  }
}

}  // namespace

// The ordering buffer is allocated once, for the largest batch that is
// sorted (kMaxRankB histograms, 256 KiB), so no fit_batch call allocates,
// frees or synchronises, and a graph captured earlier keeps a valid pointer.
hipError_t fit_scratch_init(FitScratch* s) {
  hipError_t e = hipMalloc(&s->counters, 256);
  if (e != hipSuccess) return e;
  e = hipMalloc(&s->order, sizeof(int32_t) * static_cast<size_t>(kMaxRankB));
  if (e != hipSuccess) return e;
  s->cap = kMaxRankB;
  return hipMemset(s->counters, 0, 256);
}

void fit_scratch_free(FitScratch* s) {
  if (s->order) (void)hipFree(s->order);
  if (s->counters) (void)hipFree(s->counters);
  s->order = nullptr;
  s->counters = nullptr;
  s->cap = 0;
}

int fit_max_cache_bins(int n_gauss, int bkg, int obj, int block) {
  FitLaunchFn fn = pick_fit(n_gauss, bkg, obj, block);
  int m = 0;
  if (!fn || fn(FitArgs{}, FIT_ASK_CACHE, nullptr, &m) != hipSuccess) return 0;
  return m > 0 ? m : 0;
}

int fit_max_wave_bins(int n_gauss, int bkg, int obj, int block) {
  FitLaunchFn fn = pick_fit(n_gauss, bkg, obj, block);
  int m = 0;
  if (!fn || fn(FitArgs{}, FIT_ASK_WAVES, nullptr, &m) != hipSuccess) return 0;
  return m > 0 ? m : 0;
}

// Workgroups of a full launch: no more than are resident at once.  One that
// starts when others end would still have its first place to do, one of the
// longest histograms, or in a batch that is not sorted (no more histograms than
// workgroups) any of them.  (512 histograms of 256..20,000 bins, 512 threads,
// of which one workgroup fits a CU: 156 us without the limit, 127 with it.)
static int workgroups(FitLaunchFn fn, const FitArgs& a, int num_cu, FitScratch* s) {
  const FitScratch::Launch key{reinterpret_cast<const void*>(fn), a.cache_bins, a.wave_bins};
  auto it = s->resident.find(key);
  if (it == s->resident.end()) {
    int n = 0;
    if (fn(a, FIT_ASK_RESIDENT, nullptr, &n) != hipSuccess || n < 1) n = 1;
    it = s->resident.emplace(key, n).first;
  }
  return num_cu * std::min(s->wg_per_cu, it->second);
}

// wave_bins of a context set to HF_WAVE_AUTO.  One wave per histogram saves
// the workgroup barriers and gives a CU eight fits at once, but each of these
// fits takes longer, which shows when there are few: so for batches of at
// least half as many histograms as the launch has waves, and up to 2048 bins,
// less where their slots in LDS would leave fewer workgroups resident.
// Measured with 512 workgroups of 256 threads (off, on; us): 16,384 of
// 128..1024 bins 1574, 572; 2048 of 1000 bins 254, 146; 1500 of three
// Gaussians on 256..2000 bins 477, 292; 1024 of 1000 bins 155, 136; 4096 of
// 256..65536 bins 1010, 944; 1000 of those 489, 486; but 400 of 10,000 bins
// (all sorted, none small) 173, 183, and 256 of 1000 bins 70, 96.
static int auto_wave_bins(FitLaunchFn fn, int n_gauss, int bkg, FitArgs a, int num_cu, FitScratch* s) {
  constexpr int kWaveBins = 2048, kStep = 256;
  const int groups = workgroups(fn, a, num_cu, s);
  const int waves = std::min(a.B, groups) * (s->block / 64);
  if (a.B > kMaxRankB || a.B < waves / 2) return 0;
  for (a.wave_bins = std::min(kWaveBins, fit_max_wave_bins(n_gauss, bkg, a.obj, s->block));
       a.wave_bins > 0; a.wave_bins -= kStep)
    if (workgroups(fn, a, num_cu, s) >= groups) return a.wave_bins;
  return 0;
}

hipError_t launch_fit(int n_gauss, int bkg, FitArgs a, int num_cu, FitScratch* s, hipStream_t st) {
  FitLaunchFn fn = pick_fit(n_gauss, bkg, a.obj, s->block);
  if (!fn) return hipErrorNotSupported;
  a.cache_bins = s->cache_bins;
  a.wave_bins = 0;
  a.wave_bins = s->wave_bins != kWaveAuto ? s->wave_bins : auto_wave_bins(fn, n_gauss, bkg, a, num_cu, s);
  const int grid = std::min(a.B, workgroups(fn, a, num_cu, s));
  // batches above kMaxRankB run in index order, and so do those of which
  // every workgroup takes one (the order could change nothing)
  a.sorted = (a.B <= kMaxRankB && a.B <= s->cap && (grid < a.B || a.wave_bins > 0)) ? 1 : 0;
  a.order = s->order;
  a.counters = s->counters;
  if (a.sorted) {
    hipLaunchKernelGGL(k_sort_sizes, dim3(1), dim3(kSortThreads), 0, st, a.offsets, a.B,
                       static_cast<int64_t>(a.wave_bins), a.order);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return fn(a, grid, st, nullptr);
}

}  // namespace hf
