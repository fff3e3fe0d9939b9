// mc_adjoint.hip -- reverse-time adjoint of the membrane-potential loss with
// respect to every synaptic weight, spike pattern held fixed.
//
// Loss over a window of S steps starting at step n0:
//   L = 1/(N S) sum_i sum_{n0 <= n < n0+S} (y_i(n+1) - y*)^2 .
// With the step types frozen (free / spike / refractory), the step map
// (y, I) -> (y', I') is linear: free y' = P22 y + P21 I, spike y' = y_reset,
// refractory y' = y, and always I' = P11 I + x_n.  Its transpose runs
// backwards per neuron:
//   lam  = Ly(n+1) + c (y(n+1) - y*),  c = 2/(N S)
//   LI(n) = P11 LI(n+1) + [free] P21 lam
//   Ly(n) = P22 lam | 0 | lam            (free | spike | refractory)
// with LI = Ly = 0 after the window.  The weight w_s (pA) of a synapse i -> j
// with delay d enters x_j(t + d) for each spike of i at step t, so
// dL/dw_s = sum over those spikes of LI_j(t + d + 1) (terms with
// t + d + 1 > n0 + S - 1 vanish).  The paper's explicit per-synapse weights
// (Discussion: synaptic plasticity needs them) are what make this gradient a
// per-synapse quantity.
//
// Memory: the forward keeps (y, I, r, ring) every K steps.  Segments are then
// processed last to first.  For segment [a, a+len):
//   1. (k_adj_seed)    x_seg[j][i] <- pending input of step a+j from the
//                      checkpointed ring (spikes before a) plus the redrawn
//                      drive of step a+j, every step at once;
//   2. (k_replay)      the recorded spikes of steps [a, a+len-1) add their
//                      weights into x_seg (integer sums: the same inputs the
//                      forward saw); both only where the forward has not
//                      recorded its input;
//   3. k_adj_segment   one thread per neuron: re-runs the len steps from the
//                      checkpoint (exact integration, bit-identical to the
//                      forward), keeps y and the step type of every step,
//                      then runs the transposed recurrence backwards over the
//                      segment, writing LI into a ring of R slots.  The
//                      thread's own chain bounds it (a network of 7,717
//                      neurons is 121 wavefronts), so it loads kAhead steps at
//                      once;
//   4. k_adj_verify    every recorded spike of the segment must be a spike
//                      of the recompute (and the counts must agree);
//   5. k_adj_gather    one wavefront per (source, chunk of 256 of its row): for
//                      every synapse, adds LI_tgt(t + d + 1) over the
//                      source's spikes t in [a-2, a+len-2), latest first,
//                      into grad[s] (FP64, or FP32 as g = f32(g + f32(LI))).
// Segments go latest first and each segment's spikes latest first, so every
// synapse accumulates its terms in decreasing spike time.
#pragma clang fp contract(off)

#include "mc_lif.h"

namespace mc {

constexpr int kAdjBlock = 256;

// x_seg[j][i] for j in [0, rows): the checkpointed ring's slot for step a+j
// (j < ring slots), else 0; and for j < len the drive of step a+j.  One thread
// per quad (one Philox block) and step.  (Drawn inside k_adj_segment, one
// word of a block per neuron and step in a row, the drive was most of its time.)
__global__ __launch_bounds__(kAdjBlock) void k_adj_seed(DevNet p, long long* xseg, const long long* ring_ckpt, long long a,
                                                        int len) {
  __shared__ uint64_t s_table[kMaxPops * kTableLen];
  for (int k = threadIdx.x; k < p.n_pops * kTableLen; k += blockDim.x) s_table[k] = p.table[k];
  __syncthreads();
  const long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (q >= p.n_quads) return;
  long long x[4] = {0, 0, 0, 0};
  if (j < kRingSlots) {
    const long long* slot = ring_ckpt + (size_t)((a + j) & kRingMask) * p.ring_stride + 4 * q;
    const longlong2 u = *reinterpret_cast<const longlong2*>(slot), v = *reinterpret_cast<const longlong2*>(slot + 2);
    x[0] = u.x; x[1] = u.y; x[2] = v.x; x[3] = v.y;
  }
  if (j < len) {
    const uint32_t pops = p.qpops[q];
    const U64x4 v = philox4x64_10((uint64_t)(a + j), (uint64_t)p.qlocal[q], 0, kTagDrive, p.qseed[q], 0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const unsigned pop = (pops >> (8 * k)) & 0xFFu;
      if (pop != 0xFFu) x[k] += (long long)poisson_from_u32(s_table + pop * kTableLen, hi32(pick(v, k))) * p.jext_q;
    }
  }
  long long* out = xseg + (size_t)j * p.ring_stride + 4 * q;
  *reinterpret_cast<longlong2*>(out) = make_longlong2(x[0], x[1]);
  *reinterpret_cast<longlong2*>(out + 2) = make_longlong2(x[2], x[3]);
}

constexpr int kAhead = 16;         // steps loaded at once

__global__ __launch_bounds__(kAdjBlock) void k_adj_segment(DevNet p, AdjSeg s) {
  __shared__ unsigned s_cnt;
  if (threadIdx.x == 0) s_cnt = 0;
  __syncthreads();

  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const long long st = p.ring_stride;
  unsigned spikes = 0;
  const unsigned pop = (i < p.n_pad) ? ((p.qpops[i >> 2] >> (8 * (i & 3))) & 0xFFu) : 0xFFu;
  if (pop != 0xFFu) {
    // forward recompute of the segment
    double y = s.ck_y[i], I = s.ck_I[i];
    int r = s.ck_r[i];
    for (int j0 = 0; j0 < s.len; j0 += kAhead) {
      long long x[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) x[u] = (j0 + u < s.len) ? s.xseg[(size_t)(j0 + u) * st + i] : 0;
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        if (j0 + u >= s.len) break;
        uint8_t type;
        if (lif_step(p, y, I, r, x[u], type)) ++spikes;
        s.rec_y[(size_t)(j0 + u) * st + i] = y;
        s.rec_t[(size_t)(j0 + u) * st + i] = type;
      }
    }
    // transposed recurrence, latest step first
    double ly = s.carry_ly[i], li = s.carry_li[i], loss = 0.0;
    for (int j0 = s.len - 1; j0 >= 0; j0 -= kAhead) {
      double yv[kAhead];
      uint8_t tv[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        yv[u] = (j0 - u >= 0) ? s.rec_y[(size_t)(j0 - u) * st + i] : 0.0;
        tv[u] = (j0 - u >= 0) ? s.rec_t[(size_t)(j0 - u) * st + i] : kTypePad;
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        if (j0 - u < 0) break;
        const double e = yv[u] - s.ystar;
        loss = loss + e * e;
        const double g = s.c * e;
        const double lam = ly + g;
        double li_new = p.P11 * li;
        if (tv[u] == kTypeFree) {
          li_new = li_new + p.P21 * lam;
          ly = p.P22 * lam;
        } else if (tv[u] == kTypeSpike) {
          ly = 0.0;
        } else {
          ly = lam;
        }
        li = li_new;
        s.li_ring[(size_t)((s.a + j0 - u) & (s.R - 1)) * st + i] = li;
      }
    }
    s.carry_ly[i] = ly;
    s.carry_li[i] = li;
    s.loss_part[i] = s.loss_part[i] + loss;
  }
  if (spikes) atomicAdd(&s_cnt, spikes);
  __syncthreads();
  if (threadIdx.x == 0 && s_cnt) atomicAdd(s.spike_count, (unsigned long long)s_cnt);
}

// Every recorded spike (t, i) of the segment must be a spike step of the recompute.
__global__ __launch_bounds__(kAdjBlock) void k_adj_verify(const int2* spikes, int n, const uint8_t* rec_t,
                                                          long long stride, long long a, unsigned* mismatch) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int2 sp = spikes[k];
  if (rec_t[(size_t)(sp.x - a) * stride + sp.y] != kTypeSpike) atomicAdd(mismatch, 1u);
}

constexpr int kGatherChunk = 256;   // synapses per work item (4 per lane)

// Work item it: chunk it - first[j] of source j, the j with first[j] <= it
// < first[j+1]; srcs[j] = (padded source id, first spike time in `times`,
// number of its spike times, -).  A wavefront takes consecutive items and
// finds the source of the first by search, of the others by walking on (a
// search per item was a chain of 13 dependent loads before its 256 synapses),
// and has the loads of all four synapses of a lane in flight.
template <typename G>
__global__ __launch_bounds__(kAdjBlock) void k_adj_gather(const int4* srcs, const long long* first, int nsrc,
                                                          long long n_items, const int* times, const int64_t* row_ptr,
                                                          const int32_t* tgt, const uint8_t* dly,
                                                          const double* li_ring, long long stride, int R,
                                                          long long last_m, G* grad) {
  constexpr int U = kGatherChunk / 64;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)((blockIdx.x * (long long)blockDim.x + threadIdx.x) >> 6));
  const long long nwaves = ((long long)gridDim.x * blockDim.x) >> 6;
  const long long each = (n_items + nwaves - 1) / nwaves;
  const long long it0 = wave * each, it1 = min(it0 + each, n_items);
  if (it0 >= it1) return;
  int lo = 0, hi = nsrc;
  while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (first[mid] <= it0) lo = mid; else hi = mid; }
  long long next = first[lo + 1], base = first[lo];
  int4 w = srcs[lo];
  long long r0 = row_ptr[w.x], r1 = row_ptr[w.x + 1];
  for (long long it = it0; it < it1; ++it) {
    while (it >= next) {                   // (sources without a chunk are skipped)
      ++lo;
      base = next;
      next = first[lo + 1];
      w = srcs[lo];
      r0 = row_ptr[w.x];
      r1 = row_ptr[w.x + 1];
    }
    const long long e0 = r0 + (it - base) * kGatherChunk + lane;
    int j[U], d[U];
    G acc[U];
    bool hit[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long e = e0 + u * 64;
      const bool in = e < r1;
      j[u] = in ? tgt[e] : 0;
      d[u] = in ? (int)dly[e] : (1 << 24);     // (beyond any window)
      acc[u] = in ? grad[e] : (G)0;
      hit[u] = false;
    }
    for (int q = 0; q < w.z; ++q) {
      const long long t1 = (long long)times[w.y + q] + 1;
      double v[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const long long m = t1 + d[u];
        ok[u] = m <= last_m && d[u] < (1 << 24);
        v[u] = ok[u] ? li_ring[(size_t)(m & (R - 1)) * stride + j[u]] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (ok[u]) {
          acc[u] = (G)(acc[u] + (G)v[u]);
          hit[u] = true;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (hit[u]) grad[e0 + u * 64] = acc[u];
  }
}

// First entry of row i with a target at or beyond n_pad q / kAdjRanges, for
// q <= kAdjRanges, relative to the row (rows are sorted by target).
__global__ __launch_bounds__(kAdjBlock) void k_adj_bounds(const int64_t* row_ptr, const int32_t* tgt, long long n_pad,
                                                          unsigned* rb) {
  const long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (k >= n_pad * (kAdjRanges + 1)) return;
  const long long i = k / (kAdjRanges + 1), key = n_pad * (k - i * (kAdjRanges + 1)) / kAdjRanges;
  long long lo = row_ptr[i], hi = row_ptr[i + 1];
  while (lo < hi) { const long long mid = (lo + hi) >> 1; if (tgt[mid] < key) lo = mid + 1; else hi = mid; }
  rb[k] = (unsigned)(lo - row_ptr[i]);
}

// The gather of a network whose LI values do not fit an L2: workgroup b (on
// XCD b mod 8) takes target range b mod 8 of every source, sources in the order
// of their first spike, so that what an XCD reads at a time -- its eighth of
// the targets, the ~35 steps its wavefronts are at plus the bulk of the delays
// -- is about its 4 MB of L2.  In the plain gather each 8-byte value comes as a
// line of its own from the memory side.  A wavefront takes whole sub-rows, and
// the launch has 3/4 of the wavefronts a CU holds: more widen the span of
// steps.  Full microcircuit, 100-step segments: 439 -> 340-370 us on average.
// Launches of a few steps each, to bound the span harder, left too few
// sub-rows per launch: 690 us per segment.
template <typename G>
__global__ __launch_bounds__(kAdjBlock) void k_adj_gather_xcd(const int4* srcs, int nsrc, const int* times,
                                                              const int64_t* row_ptr, const unsigned* rb,
                                                              const int32_t* tgt, const uint8_t* dly,
                                                              const double* li_ring, long long stride, int R,
                                                              long long last_m, G* grad) {
  constexpr int U = kGatherChunk / 64;
  const int lane = threadIdx.x & 63, range = blockIdx.x % kAdjRanges;
  const int wave = __builtin_amdgcn_readfirstlane((int)((blockIdx.x / kAdjRanges) * (kAdjBlock / 64) + (threadIdx.x >> 6)));
  const int nwaves = (int)(gridDim.x / kAdjRanges) * (kAdjBlock / 64);
  for (int k = wave; k < nsrc; k += nwaves) {
    const int4 w = srcs[k];
    const unsigned* b = rb + (size_t)w.x * (kAdjRanges + 1) + range;
    const long long r = row_ptr[w.x], r1 = r + b[1];
    for (long long e0 = r + b[0] + lane; e0 - lane < r1; e0 += kGatherChunk) {
      int j[U], d[U];
      G acc[U];
      bool hit[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const long long e = e0 + u * 64;
        const bool in = e < r1;
        j[u] = in ? tgt[e] : 0;
        d[u] = in ? (int)dly[e] : (1 << 24);   // (beyond any window)
        acc[u] = in ? grad[e] : (G)0;
        hit[u] = false;
      }
      for (int q = 0; q < w.z; ++q) {
        const long long t1 = (long long)times[w.y + q] + 1;
        double v[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const long long m = t1 + d[u];
          ok[u] = m <= last_m && d[u] < (1 << 24);
          v[u] = ok[u] ? li_ring[(size_t)(m & (R - 1)) * stride + j[u]] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (ok[u]) {
            acc[u] = (G)(acc[u] + (G)v[u]);
            hit[u] = true;
          }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (hit[u]) grad[e0 + u * 64] = acc[u];
    }
  }
}

// ---------------------------------------------------------------------------
// host wrappers
// ---------------------------------------------------------------------------
hipError_t launch_adj_seed(const DevNet& p, long long* xseg, const long long* ring_ckpt, long long a, int len, int rows,
                           hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const dim3 grid((unsigned)((p.n_quads + kAdjBlock - 1) / kAdjBlock), (unsigned)rows);
  hipLaunchKernelGGL(k_adj_seed, grid, dim3(kAdjBlock), 0, s, p, xseg, ring_ckpt, a, len);
  return hipGetLastError();
}

hipError_t launch_adj_segment(const DevNet& p, const AdjSeg& a, hipStream_t s) {
  const unsigned grid = (unsigned)((p.n_pad + kAdjBlock - 1) / kAdjBlock);
  hipLaunchKernelGGL(k_adj_segment, dim3(grid), dim3(kAdjBlock), 0, s, p, a);
  return hipGetLastError();
}

hipError_t launch_adj_verify(const int2* spikes, int n, const uint8_t* rec_t, long long stride, long long a,
                             unsigned* mismatch, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_adj_verify, dim3((unsigned)((n + kAdjBlock - 1) / kAdjBlock)), dim3(kAdjBlock), 0, s, spikes,
                     n, rec_t, stride, a, mismatch);
  return hipGetLastError();
}

hipError_t launch_adj_gather(const int4* srcs, const long long* first, int nsrc, long long n_items, const int* times,
                             const int64_t* row_ptr, const int32_t* tgt, const uint8_t* dly, const double* li_ring,
                             long long stride, int R, long long last_m, void* grad, bool fp32, int grid, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  if (fp32)
    hipLaunchKernelGGL(k_adj_gather<float>, dim3(grid), dim3(kAdjBlock), 0, s, srcs, first, nsrc, n_items, times,
                       row_ptr, tgt, dly, li_ring, stride, R, last_m, (float*)grad);
  else
    hipLaunchKernelGGL(k_adj_gather<double>, dim3(grid), dim3(kAdjBlock), 0, s, srcs, first, nsrc, n_items, times,
                       row_ptr, tgt, dly, li_ring, stride, R, last_m, (double*)grad);
  return hipGetLastError();
}

// The ranged gather pays where the LI values of the steps in flight (~60: the
// wavefronts' span and the bulk of the delays) do not fit one 4 MB L2 as they
// are; below, sub-rows of an eighth only leave lanes idle.
bool adj_gather_ranged(long long stride) { return stride * 8 * 60 > (4ll << 20); }

hipError_t launch_adj_bounds(const int64_t* row_ptr, const int32_t* tgt, long long n_pad, unsigned* rb, hipStream_t s) {
  const long long n = n_pad * (kAdjRanges + 1);
  hipLaunchKernelGGL(k_adj_bounds, dim3((unsigned)((n + kAdjBlock - 1) / kAdjBlock)), dim3(kAdjBlock), 0, s, row_ptr, tgt,
                     n_pad, rb);
  return hipGetLastError();
}

hipError_t launch_adj_gather_xcd(const int4* srcs, int nsrc, const int* times, const int64_t* row_ptr, const unsigned* rb,
                                 const int32_t* tgt, const uint8_t* dly, const double* li_ring, long long stride, int R,
                                 long long last_m, void* grad, bool fp32, int n_cu, hipStream_t s) {
  if (nsrc <= 0) return hipSuccess;
  const int grid = n_cu * 6 / kAdjRanges * kAdjRanges + kAdjRanges;
  if (fp32)
    hipLaunchKernelGGL(k_adj_gather_xcd<float>, dim3(grid), dim3(kAdjBlock), 0, s, srcs, nsrc, times, row_ptr, rb, tgt, dly,
                       li_ring, stride, R, last_m, (float*)grad);
  else
    hipLaunchKernelGGL(k_adj_gather_xcd<double>, dim3(grid), dim3(kAdjBlock), 0, s, srcs, nsrc, times, row_ptr, rb, tgt, dly,
                       li_ring, stride, R, last_m, (double*)grad);
  return hipGetLastError();
}

}  // namespace mc
