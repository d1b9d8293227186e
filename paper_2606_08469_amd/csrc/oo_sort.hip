// Spatial bucketing of the residual step's queries.
//
// The query kernel's cost is dominated by the texel gathers of the fine
// levels, whose tables (hundreds of MB) miss in the caches when queries come
// in sampling order. Grouping queries by a coarse octree cell before they
// are evaluated makes neighbouring query tiles read the same nodes' maps, so
// those lines are fetched once and then hit in L2. The grouping is a counting
// sort by the Morton code of the query's cell at octree level c = min(D, 4),
// with the secondary queries (q >= n_lhs) in a second key range, so the
// first n_lhs sorted positions are exactly the LHS queries the backward
// walks. The order inside a bucket is not fixed (LDS atomics hand out
// slots), which only changes the summation order of the gradients.
//
// Three passes over Q queries split into NB contiguous chunks:
//   1. per-chunk histograms in LDS          -> counts[NB][K]
//   2. per-bucket exclusive prefix over the chunks, bucket totals, and the
//      exclusive scan of the totals          -> counts (in place), start[K]
//   3. each chunk hands out slots from LDS cursors: order[pos] = q (the
//      query at sorted position pos) and rank[q] = pos.
// Only 4-byte indices move: the kernels that evaluate the sorted queries
// read positions and directions through order, and the residual assembly
// reads the sorted radiance through rank.
//
// With a disparity predictor a fourth pass refines the order (fine): pass 3
// writes pairs (q, key at level min(D, c + 2)) instead, and each workgroup
// sorts a run of 8192 consecutive pairs by that key. Neighbouring lanes then
// read the same lines of the fine hash levels, whose requests to the L2 bound
// the predictor (2.2 million queries: 667 us before, 529 after; the shifted
// encode 806 and 755; the pass itself takes 42, most of it for writing rank
// out of order).
#include <hip/hip_runtime.h>

#include "oo_device.h"
#include "oo_internal.h"

namespace oo {

constexpr int kSortThreads = 1024;
constexpr int kSortMaxChunks = 256;
// The finer order pays where a wave's 64 queries then share lines of the hash
// tables: with the disparity predictor (16 levels of gathers per query) and
// enough queries. Whole training steps with it and without: 147,456 queries
// 776 us and 771, 540,672 queries 1076 and 1094, 2.2 million 2680 and 2806.
// Without the predictor the query kernel gains as much as the sort costs
// (9.4 million queries: 1206 us and 41 more for the sort, 1278 without).
constexpr int64_t kFineMin = 1 << 18;


// Sort key of query q: the Morton code of its cell at level F, with the
// secondary queries behind the others. key >> 3 (F - c) is its bucket.
__device__ inline int sort_key(const float x[3], int D, int F, int64_t q, int64_t n_lhs) {
  const int sh = D - F;
  const int cx = quant_axis(x[0], D) >> sh, cy = quant_axis(x[1], D) >> sh, cz = quant_axis(x[2], D) >> sh;
  int code = 0;
  for (int b = 0; b < F; ++b)
    code |= (((cx >> b) & 1) | (((cy >> b) & 1) << 1) | (((cz >> b) & 1) << 2)) << (3 * b);
  return code + (q >= n_lhs ? (1 << (3 * F)) : 0);
}

__global__ __launch_bounds__(kSortThreads) void sort_hist_kernel(const QuerySrc src, int64_t Q, int64_t n_lhs, int D,
                                                                 int c, int K, int64_t chunk,
                                                                 int32_t* __restrict__ counts) {
  extern __shared__ int hist[];
  for (int b = threadIdx.x; b < K; b += blockDim.x) hist[b] = 0;
  __syncthreads();
  const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < Q ? lo + chunk : Q;
  for (int64_t q = lo + threadIdx.x; q < hi; q += blockDim.x) {
    float x[3];
    load_pos(src, q, x);
    atomicAdd(&hist[sort_key(x, D, c, q, n_lhs)], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < K; b += blockDim.x) counts[(int64_t)blockIdx.x * K + b] = hist[b];
}

// Exclusive prefix of each bucket's counts over the chunks (in place) and the
// bucket totals. Four waves share 64 buckets, a quarter of the chunks each,
// so that all counts are in flight at once (one thread per bucket, 16 counts
// at a time: 20 us for 256 chunks of 8192 buckets; this takes 8).
constexpr int kScanPer = kSortMaxChunks / 4;
__global__ __launch_bounds__(256) void sort_colscan_kernel(int32_t* __restrict__ counts, int NB, int K,
                                                           int32_t* __restrict__ total) {
  __shared__ int sums[4][64];
  const int lane = threadIdx.x & 63, part = threadIdx.x >> 6, b = blockIdx.x * 64 + lane;
  const int w0 = part * kScanPer;
  int v[kScanPer], s = 0;
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) v[j] = b < K && w0 + j < NB ? counts[(int64_t)(w0 + j) * K + b] : 0;
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) s += v[j];
  sums[part][lane] = s;
  __syncthreads();
  if (b >= K) return;
  int run = 0;
  for (int p = 0; p < part; ++p) run += sums[p][lane];
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    if (w0 + j < NB) counts[(int64_t)(w0 + j) * K + b] = run;
    run += v[j];
  }
  if (part == 3) total[b] = run;
}

// One workgroup: start[b] = sum of total[0 .. b-1], up to kStartPer
// consecutive buckets per thread, summed over the wave by shuffles (9 us for
// 8192 buckets; a scan in LDS with two barriers per step took 13).
constexpr int kStartPer = 8;
__global__ __launch_bounds__(1024) void sort_start_kernel(const int32_t* __restrict__ total, int K,
                                                          int32_t* __restrict__ start) {
  __shared__ int wsum[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int per = (K + 1023) / 1024, b0 = threadIdx.x * per;
  int v[kStartPer], s = 0;
#pragma unroll
  for (int j = 0; j < kStartPer; ++j) v[j] = j < per && b0 + j < K ? total[b0 + j] : 0;
#pragma unroll
  for (int j = 0; j < kStartPer; ++j) s += v[j];
  int run = s;
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_up(run, off);
    if (lane >= off) run += t;
  }
  if (lane == 63) wsum[wave] = run;
  __syncthreads();
  run -= s;
  for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
  for (int j = 0; j < kStartPer; ++j)
    if (j < per && b0 + j < K) {
      start[b0 + j] = run;
      run += v[j];
    }
}

// FINE: pairs (q, key) for sort_fine_kernel in place of the order itself.
template <bool FINE>
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(const QuerySrc src, int64_t Q, int64_t n_lhs,
                                                                    int D, int c, int F, int K, int64_t chunk,
                                                                    const int32_t* __restrict__ prefix,
                                                                    const int32_t* __restrict__ start,
                                                                    int32_t* __restrict__ order,
                                                                    int32_t* __restrict__ rank,
                                                                    int2* __restrict__ pairs) {
  extern __shared__ int cur[];
  for (int b = threadIdx.x; b < K; b += blockDim.x) cur[b] = start[b] + prefix[(int64_t)blockIdx.x * K + b];
  __syncthreads();
  const int64_t lo = (int64_t)blockIdx.x * chunk, hi = lo + chunk < Q ? lo + chunk : Q;
  for (int64_t q = lo + threadIdx.x; q < hi; q += blockDim.x) {
    float x[3];
    load_pos(src, q, x);
    const int key = sort_key(x, D, F, q, n_lhs);
    const int pos = atomicAdd(&cur[key >> (3 * (F - c))], 1);
    if constexpr (FINE) {
      pairs[pos] = make_int2((int)q, key);
    } else {
      order[pos] = (int32_t)q;
      rank[q] = pos;
    }
  }
}

// Each workgroup sorts a run of kFineRun positions by the finer key: the run
// is in bucket order already, so its buckets are numbered by counting the
// changes, and (number, fine part) is the key of a counting sort in LDS.
// Buckets past the kFineRanks'th keep their positions. No query leaves its
// bucket, so the LHS queries stay in front.
constexpr int kFinePer = 8;
constexpr int kFineRun = kSortThreads * kFinePer;
constexpr int kFineRanks = 64;
constexpr int kFineBits = 6;  // two levels
__global__ __launch_bounds__(kSortThreads) void sort_fine_kernel(const int2* __restrict__ pairs, int64_t Q,
                                                                 int fine_bits, int32_t* __restrict__ order,
                                                                 int32_t* __restrict__ rank) {
  constexpr int NC = kFineRanks << kFineBits, W = kSortThreads / 64;
  __shared__ int cnt[NC], changes[kFinePer * W], out[kFineRun], wsum[W];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)blockIdx.x * kFineRun;
  int2 e[kFinePer];
#pragma unroll
  for (int j = 0; j < kFinePer; ++j) {
    const int64_t p = base + j * kSortThreads + tid;
    e[j] = p < Q ? pairs[p] : make_int2(-1, 0);
  }
#pragma unroll
  for (int i = 0; i < NC / kSortThreads; ++i) cnt[tid + i * kSortThreads] = 0;
  uint64_t change[kFinePer];
#pragma unroll
  for (int j = 0; j < kFinePer; ++j) {
    const int64_t p = base + j * kSortThreads + tid;
    int before = __shfl_up(e[j].y, 1);
    if (lane == 0) before = p > base && p < Q ? pairs[p - 1].y : e[j].y;
    change[j] = __ballot(e[j].x >= 0 && (before >> fine_bits) != (e[j].y >> fine_bits));
    if (lane == 0) changes[j * W + wave] = __popcll(change[j]);
  }
  __syncthreads();
  if (wave == 0) {  // inclusive prefix of the kFinePer * W counts, two per lane
    static_assert(kFinePer * W == 128, "two counts per lane");
    const int a = changes[2 * lane], b = changes[2 * lane + 1];
    int s = a + b;
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(s, off);
      if (lane >= off) s += v;
    }
    changes[2 * lane] = s - a - b;
    changes[2 * lane + 1] = s - b;
  }
  __syncthreads();
  int key[kFinePer], slot[kFinePer];
#pragma unroll
  for (int j = 0; j < kFinePer; ++j) {
    const uint64_t upto = lane == 63 ? change[j] : change[j] & ((2ull << lane) - 1);
    const int rank = changes[j * W + wave] + __popcll(upto);
    key[j] = rank < kFineRanks ? (rank << kFineBits) | (e[j].y & ((1 << fine_bits) - 1)) : -1;
    slot[j] = e[j].x >= 0 && key[j] >= 0 ? atomicAdd(&cnt[key[j]], 1) : 0;
  }
  __syncthreads();
  {  // exclusive prefix of the counters, NC / kSortThreads consecutive ones per thread
    constexpr int per = NC / kSortThreads;
    int v[per], s = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) s += v[i] = cnt[tid * per + i];
    int inc = s;
    for (int off = 1; off < 64; off <<= 1) {
      const int t = __shfl_up(inc, off);
      if (lane >= off) inc += t;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int run = inc - s;
    for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
    for (int i = 0; i < per; ++i) {
      cnt[tid * per + i] = run;
      run += v[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kFinePer; ++j)
    if (e[j].x >= 0) out[key[j] >= 0 ? cnt[key[j]] + slot[j] : j * kSortThreads + tid] = e[j].x;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kFinePer; ++j) {
    const int i = j * kSortThreads + tid;
    if (base + i < Q) {
      order[base + i] = out[i];
      rank[out[i]] = (int32_t)(base + i);
    }
  }
}

SortShape sort_shape(int64_t Q, int D, bool fine) {
  SortShape s;
  s.c = D < 4 ? D : 4;
  s.K = 2 << (3 * s.c);  // at most 1024 kStartPer
  s.F = !fine || Q < kFineMin ? s.c : (D < s.c + 2 ? D : s.c + 2);
  int64_t nb = (Q + kSortThreads - 1) / kSortThreads;
  s.NB = (int)(nb < 1 ? 1 : (nb > kSortMaxChunks ? kSortMaxChunks : nb));
  s.chunk = (Q + s.NB - 1) / s.NB;
  return s;
}

hipError_t launch_spatial_sort(const QuerySrc& src, int64_t Q, int64_t n_lhs, int D, int32_t* counts, int32_t* total,
                               int32_t* start, int32_t* order, int32_t* rank, void* scratch, bool fine,
                               hipStream_t st) {
  if (Q == 0) return hipSuccess;
  const SortShape s = sort_shape(Q, D, fine);
  const size_t lds = (size_t)s.K * sizeof(int);
  hipLaunchKernelGGL(sort_hist_kernel, dim3(s.NB), dim3(kSortThreads), lds, st, src, Q, n_lhs, D, s.c, s.K, s.chunk,
                     counts);
  hipLaunchKernelGGL(sort_colscan_kernel, dim3((s.K + 63) / 64), dim3(256), 0, st, counts, s.NB, s.K, total);
  hipLaunchKernelGGL(sort_start_kernel, dim3(1), dim3(1024), 0, st, total, s.K, start);
  if (s.F > s.c) {
    int2* const pairs = reinterpret_cast<int2*>(scratch);
    hipLaunchKernelGGL(sort_scatter_kernel<true>, dim3(s.NB), dim3(kSortThreads), lds, st, src, Q, n_lhs, D, s.c, s.F,
                       s.K, s.chunk, counts, start, order, rank, pairs);
    hipLaunchKernelGGL(sort_fine_kernel, dim3((unsigned)((Q + kFineRun - 1) / kFineRun)), dim3(kSortThreads), 0, st,
                       pairs, Q, 3 * (s.F - s.c), order, rank);
  } else {
    hipLaunchKernelGGL(sort_scatter_kernel<false>, dim3(s.NB), dim3(kSortThreads), lds, st, src, Q, n_lhs, D, s.c, s.F,
                       s.K, s.chunk, counts, start, order, rank, nullptr);
  }
  return hipGetLastError();
}

}  // namespace oo
