// mc_raster.hip -- read-back of the spike raster, ordered on the device.
//
// Every workgroup of the simulation kernels appends its spikes to a raster
// segment of its own (no global atomic), by step; the caller gets them sorted
// by step, then neuron id.  Sorting on the host took most of a batch's call
// (650,000 spikes of 64 instances: 44 of 71 ms, one map from padded to dense
// id and one comparison sort per step), and four copies with three
// synchronisations most of a short call (100 of 145 us for one step of the
// balanced network).  Here the device orders the spikes and writes them into
// pinned host memory; the host waits once for a short span and twice for a
// long one.
//
// Up to kSmall spikes one workgroup does all: prefix sums of the segments'
// lengths, gather, bitonic sort of (step, id) keys in LDS, which for the few
// hundred spikes of a short call is a handful of microseconds.  More are
// counted per step, scattered into their step's bucket and sorted there, a
// workgroup per step: by rank for a few, else through a bitmap over the ids (a
// neuron spikes at most once per step), whose cost does not depend on the
// number of spikes.
#include <algorithm>

#include "mc_device.h"

namespace mc {

namespace {

constexpr int kSmall = kRasterSmall;
constexpr int kSmallBlock = 1024;
constexpr int kMaxSeg = 4096;              // segments whose prefix fits the small path's LDS
constexpr int kStepBlock = 256;
constexpr int kRank = 256;                 // spikes of a step sorted by rank
constexpr int kMapIds = 1 << 18;           // ids per bitmap pass (32 KB of LDS: several steps per compute unit)

// Dense id of padded id i: instances start at inst_pad[b] and inst_off[b].
__device__ __forceinline__ int dense_id(const RasterArgs& a, int i) {
  int lo = 0, hi = a.n_inst;               // inst_pad[lo] <= i < inst_pad[hi]
  while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (a.inst_pad[mid] <= i) lo = mid; else hi = mid; }
  return i - (int)(a.inst_pad[lo] - a.inst_off[lo]);
}

// Block-wide exclusive scan of one int per thread; every thread gets the total.
template <int kBlock>
__device__ __forceinline__ int scan_block(int v, int* s_tmp, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  __syncthreads();
  if (lane == 63) s_tmp[wave] = x;
  __syncthreads();
  int before = 0, all = 0;
  for (int w = 0; w < kBlock / 64; ++w) { const int t = s_tmp[w]; before += (w < wave) ? t : 0; all += t; }
  *total = all;
  return before + x - v;
}

}  // namespace

// head[0] = spikes, head[1] = error bits, head[2] = 1 if they have been
// written; else there are too many, the caller takes the long way, and head[3]
// and head[4] are their first and last step.  The range comes from the spikes:
// a graph that the program captured may have run any number of steps since the
// last read-back.
__global__ __launch_bounds__(kSmallBlock) void k_raster_small(RasterArgs a) {
  __shared__ int s_pre[kMaxSeg + 1];
  __shared__ unsigned long long s_key[kSmall];
  __shared__ int s_tmp[kSmallBlock / 64];
  const int tid = threadIdx.x;
  const int per = (a.n_seg + kSmallBlock - 1) / kSmallBlock;   // segments per thread
  long long mine = 0;
  for (int k = tid * per; k < min((tid + 1) * per, a.n_seg); ++k) mine += a.cnt[k];
  // (a count beyond int is beyond kSmall too)
  int total = 0;
  const bool big = __syncthreads_or(mine > (long long)(1 << 20));
  int at = scan_block<kSmallBlock>(big ? 0 : (int)mine, s_tmp, &total);
  const bool small = !big && total <= kSmall && a.n_seg <= kMaxSeg;
  if (!small) {
    // the long way needs the exact total
    unsigned long long* sum = reinterpret_cast<unsigned long long*>(s_key);
    int* range = reinterpret_cast<int*>(s_key + 1);
    if (tid == 0) { sum[0] = 0; range[0] = 0x7FFFFFFF; range[1] = -1; }
    __syncthreads();
    int first = 0x7FFFFFFF, last = -1;
    for (int k = tid * per; k < min((tid + 1) * per, a.n_seg); ++k) {
      const long long c = a.cnt[k];        // (a segment is ordered by step)
      if (c == 0) continue;
      first = min(first, a.raster[(size_t)k * a.cap].x);
      last = max(last, a.raster[(size_t)k * a.cap + c - 1].x);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      mine += __shfl_xor(mine, o, 64);
      first = min(first, __shfl_xor(first, o, 64));
      last = max(last, __shfl_xor(last, o, 64));
    }
    if ((tid & 63) == 0) {
      atomicAdd(sum, (unsigned long long)mine);
      atomicMin(&range[0], first);
      atomicMax(&range[1], last);
    }
    __syncthreads();
    if (tid == 0) {
      a.head[0] = (long long)sum[0]; a.head[1] = *a.overflow; a.head[2] = 0;
      a.head[3] = range[0]; a.head[4] = range[1];
    }
    return;
  }
  for (int k = tid * per; k < min((tid + 1) * per, a.n_seg); ++k) {
    s_pre[k] = at;
    at += (int)a.cnt[k];
  }
  if (tid == 0) s_pre[a.n_seg] = total;
  int n2 = 1;
  while (n2 < total) n2 <<= 1;
  __syncthreads();
  for (int k = tid; k < n2; k += kSmallBlock) {
    unsigned long long key = ~0ull;
    if (k < total) {
      int lo = 0, hi = a.n_seg;            // segment: s_pre[lo] <= k < s_pre[hi]
      while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (s_pre[mid] <= k) lo = mid; else hi = mid; }
      const int2 e = a.raster[(size_t)lo * a.cap + (k - s_pre[lo])];
      key = (unsigned long long)(unsigned)e.x << 32 | (unsigned)e.y;
    }
    s_key[k] = key;
  }
  for (int k = tid; k < a.n_seg; k += kSmallBlock) a.cnt[k] = 0;
  for (int size = 2; size <= n2; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      __syncthreads();
      for (int k = tid; k < n2 / 2; k += kSmallBlock) {
        const int i = 2 * k - (k & (stride - 1)), j = i + stride;
        const unsigned long long x = s_key[i], y = s_key[j];
        if ((x > y) == ((i & size) == 0)) { s_key[i] = y; s_key[j] = x; }
      }
    }
  __syncthreads();
  for (int k = tid; k < total; k += kSmallBlock) {
    a.out_step[k] = (int)(s_key[k] >> 32);
    a.out_id[k] = dense_id(a, (int)(unsigned)s_key[k]);
  }
  if (tid == 0) { a.head[0] = total; a.head[1] = *a.overflow; a.head[2] = 1; }
}

// Spikes per step: hist[step - lo].
__global__ void k_raster_hist(RasterArgs a, int* hist) {
  const long long c = a.cnt[blockIdx.x];
  const int2* src = a.raster + (size_t)blockIdx.x * a.cap;
  for (long long k = threadIdx.x; k < c; k += blockDim.x) {
    const int s = src[k].x - a.lo;
    if ((unsigned)s < (unsigned)a.span) atomicAdd(&hist[s], 1);
  }
}

// off[k] = spikes before step lo + k (k <= span); cursor[k] likewise (k < span);
// head[5] = spikes in all.
__global__ __launch_bounds__(kSmallBlock) void k_raster_scan(const int* hist, int span, int* off, int* cursor, long long* head) {
  __shared__ int s_tmp[kSmallBlock / 64];
  const int per = (int)(((long long)span + kSmallBlock - 1) / kSmallBlock);
  const int b = (int)min((long long)threadIdx.x * per, (long long)span), e = (int)min((long long)b + per, (long long)span);
  int mine = 0;
  for (int k = b; k < e; ++k) mine += hist[k];
  int total;
  int at = scan_block<kSmallBlock>(mine, s_tmp, &total);
  for (int k = b; k < e; ++k) {
    const int h = hist[k];
    off[k] = at;
    cursor[k] = at;
    at += h;
  }
  if (threadIdx.x == 0) { off[span] = total; head[5] = total; }
}

// Every spike's padded id into its step's bucket (any order).
__global__ void k_raster_scatter(RasterArgs a, int* cursor, int* bucket) {
  const long long c = a.cnt[blockIdx.x];
  const int2* src = a.raster + (size_t)blockIdx.x * a.cap;
  for (long long k = threadIdx.x; k < c; k += blockDim.x) {
    const int2 e = src[k];
    const int s = e.x - a.lo;
    if ((unsigned)s < (unsigned)a.span) bucket[atomicAdd(&cursor[s], 1)] = e.y;
  }
}

// Step lo + at, at = first + blockIdx.x: its ids in ascending order, dense, to
// out_id; the steps to out_step; the first workgroup empties the segments.
__global__ __launch_bounds__(kStepBlock) void k_raster_sort(RasterArgs a, int first, const int* off, const int* bucket,
                                                            long long n_pad) {
  __shared__ unsigned s_map[kMapIds / 32];
  __shared__ int s_tmp[kStepBlock / 64];
  const int tid = threadIdx.x, at = first + (int)blockIdx.x, b = off[at], c = off[at + 1] - b;
  if (at == 0)
    for (int k = tid; k < a.n_seg; k += kStepBlock) a.cnt[k] = 0;
  for (int k = tid; k < c; k += kStepBlock) a.out_step[b + k] = a.lo + at;
  if (c <= kRank) {
    int* s_id = reinterpret_cast<int*>(s_map);
    const int id = (tid < c) ? bucket[b + tid] : 0;
    if (tid < c) s_id[tid] = id;
    __syncthreads();
    int rank = 0;
    for (int k = 0; k < c; ++k) rank += s_id[k] < id;
    if (tid < c) a.out_id[b + rank] = dense_id(a, id);
    return;
  }
  int done = 0;
  for (long long id0 = 0; id0 < n_pad; id0 += kMapIds) {
    const int words = (int)((min((long long)kMapIds, n_pad - id0) + 31) / 32);
    __syncthreads();
    for (int k = tid; k < words; k += kStepBlock) s_map[k] = 0;
    __syncthreads();
    for (int k = tid; k < c; k += kStepBlock) {
      const long long i = bucket[b + k] - id0;
      if (i >= 0 && i < kMapIds) atomicOr(&s_map[i >> 5], 1u << (i & 31));
    }
    __syncthreads();
    const int per = (words + kStepBlock - 1) / kStepBlock;   // consecutive words per thread: ascending ids
    const int w0 = min(tid * per, words), w1 = min(w0 + per, words);
    int mine = 0;
    for (int w = w0; w < w1; ++w) mine += __popc(s_map[w]);
    int total;
    int o = done + scan_block<kStepBlock>(mine, s_tmp, &total);
    for (int w = w0; w < w1; ++w)
      for (unsigned m = s_map[w]; m; m &= m - 1)
        a.out_id[b + o++] = dense_id(a, (int)id0 + 32 * w + __builtin_ctz(m));
    done += total;
  }
}

hipError_t launch_raster_small(const RasterArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_raster_small, dim3(1), dim3(kSmallBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_raster_order(const RasterArgs& a, long long n_pad, int* hist, int* off, int* cursor, int* bucket,
                               hipStream_t s) {
  const int span = a.span;
  if (span < 1 || a.n_seg < 1) return hipErrorInvalidValue;
  hipError_t e = hipMemsetAsync(hist, 0, sizeof(int) * (size_t)span, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_raster_hist, dim3((unsigned)a.n_seg), dim3(256), 0, s, a, hist);
  hipLaunchKernelGGL(k_raster_scan, dim3(1), dim3(kSmallBlock), 0, s, hist, span, off, cursor, a.head);
  hipLaunchKernelGGL(k_raster_scatter, dim3((unsigned)a.n_seg), dim3(256), 0, s, a, cursor, bucket);
  constexpr long long kSteps = 1 << 22;      // workgroups of a launch: 2^32 threads are the most
  for (long long first = 0; first < span; first += kSteps)
    hipLaunchKernelGGL(k_raster_sort, dim3((unsigned)std::min(kSteps, span - first)), dim3(kStepBlock), 0, s, a, (int)first, off,
                       bucket, n_pad);
  return hipGetLastError();
}

}  // namespace mc
