// mc_kernels.hip -- HIP kernels of the simulation cycle for gfx950.
//
// Step n of the cycle (Fig. 1 caption of the paper: "update" integrates the
// state of the neurons, "deliver" distributes spike events to the targets):
//   drive   : Poisson count k_i(n) by inverse CDF of the upper 32 bits of
//             a Philox4x64-10 word keyed (n, local quad, 0, DRIVE);
//   update  : x = (ring[n][i] + k_i(n) J_q) 2^-16 pA, ring slot cleared;
//             free neurons y <- P22 y + P21 I (+ P20 I_e), refractory ones
//             count down; I <- P11 I + x; spike iff free and y >= theta,
//             then y <- y_reset, r <- t_ref/h   (exact integration, FP64,
//             no contraction);
//   compact : spike flags -> dense id list per workgroup, appended to the
//             raster;
//   deliver : every synapse s of every spiking row adds w_q[s] to
//             ring[(n + d_s) mod 128][tgt_s] with an int64 atomic -- integer
//             sums, so the result does not depend on the order.
// Kernels are launched one per step and replayed from a HIP graph; the
// kernel boundary is the device-wide barrier between the delivery of step
// n and the update of step n+1 (the smallest delay is one step).
#pragma clang fp contract(off)

#include "mc_lif.h"

namespace mc {

constexpr int kMaxBlock = 1024;
constexpr int kMaxQuadsPerWg = 256;             // quads updated by one workgroup of k_step

// ---------------------------------------------------------------------------
// Shared pieces
// ---------------------------------------------------------------------------

// Loads the Poisson tables of all populations into LDS.
__device__ __forceinline__ void load_tables(const DevNet& p, uint64_t* s_table) {
  for (int k = threadIdx.x; k < p.n_pops * kTableLen; k += blockDim.x) s_table[k] = p.table[k];
}

__device__ __forceinline__ uint64_t lane_swap(uint64_t v) {   // lanes 0<->1, 2<->3
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)v, 0xB1, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), 0xB1, 0xF, 0xF, true);
  return (uint64_t)hi << 32 | lo;
}

// Upper 32 bits of word (lane & 3) of philox4x64_10(n, local, 0, kTagDrive;
// seed, 0), for the four lanes of a quad together: even lanes hold the words
// 0 and 1, odd lanes 2 and 3, and each multiplies once per round and swaps the
// product with its neighbour -- half the 64-bit products of a lane that makes
// the whole block, which lie on the step's critical path.
__device__ __forceinline__ uint32_t quad_drive_word(uint64_t n, uint64_t local, uint64_t seed) {
  const bool odd = threadIdx.x & 1;
  const uint64_t mul = odd ? 0xCA5A826395121157ULL : 0xD2E7470EE14C6C93ULL;
  const uint64_t weyl = odd ? 0xBB67AE8584CAA73BULL : 0x9E3779B97F4A7C15ULL;
  uint64_t x = odd ? 0 : n, y = odd ? (uint64_t)kTagDrive : local, k = odd ? 0 : seed;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t lo = mul * x, hi = __umul64hi(mul, x);
    x = lane_swap(hi) ^ y ^ k;
    y = lane_swap(lo);
    k += weyl;
  }
  // lane 0: its x; 1: lane 0's y; 2: lane 3's x; 3: its y
  const uint64_t send = odd ? x : y, got = lane_swap(send);
  return hi32((threadIdx.x & 3) == 0 ? x : (threadIdx.x & 3) == 3 ? y : got);
}

// ---------------------------------------------------------------------------
// One step: update + compaction + owner delivery.  Workgroup g updates the
// quads [g*qpw, (g+1)*qpw), one neuron per thread and round, lists its spikes
// in LDS, appends them to its private raster segment and walks their synapse
// rows with all of its threads.
//
// A step of a small network is a chain of latencies, not work: step number,
// state, drive, spikes, rows, atomics.  So every load that does not need the
// step number or the spikes (state, row bounds, raster position) goes out
// first, the bookkeeping is atomics nobody waits for, and a row of up to 8
// entries per thread is one round of loads.
// Per step, against one quad per lane of the first wavefronts with each load
// where it is used: balanced network 10.4 -> 6.6 us, microcircuit at scale 0.3
// 17.1 -> 11.8 us, full microcircuit 34 -> 29 us (there bound by the device
// atomics of its rows).
// ---------------------------------------------------------------------------
template <bool kOwnerLists>
__global__ __launch_bounds__(kMaxBlock) void k_step(DevNet p, int offset, int qpw, int wave_rows) {
  constexpr int kRounds = 4;                    // neurons per thread at most (qpw <= threads)
  constexpr int kAhead = 8;                     // entries of a row in flight per thread
  __shared__ uint64_t s_table[kMaxPops * kTableLen];
  __shared__ int s_spk[4 * kMaxQuadsPerWg], s_len[4 * kMaxQuadsPerWg];
  __shared__ long long s_rs[4 * kMaxQuadsPerWg];
  __shared__ unsigned long long s_events;
  __shared__ int s_total;

  const int tid = threadIdx.x, nthr = blockDim.x;
  const long long j0 = (long long)blockIdx.x * 4 * qpw;
  const int nj = (int)min((long long)4 * qpw, 4 * p.n_quads - j0);
  const long long n = *p.step_base + offset;
  const long long rbase = p.raster_cnt[blockIdx.x];
  double y[kRounds], I[kRounds];
  int r[kRounds];
  uint32_t pops[kRounds];
  uint64_t local[kRounds], seed[kRounds];
  long long rs[kRounds], re[kRounds];
#pragma unroll
  for (int c = 0; c < kRounds; ++c) {
    const int jl = tid + c * nthr;
    if (c * nthr < nj && jl < nj) {
      const long long j = j0 + jl, q = j >> 2;
      pops[c] = p.qpops[q]; local[c] = (uint64_t)p.qlocal[q]; seed[c] = p.qseed[q];
      y[c] = p.y[j]; I[c] = p.I[j]; r[c] = p.r[j];
      rs[c] = p.row_ptr[j]; re[c] = p.row_ptr[j + 1];
    }
  }
  load_tables(p, s_table);
  if (tid == 0) { s_events = 0; s_total = 0; }
  __syncthreads();

  long long ck = -1;                            // adjoint forward: the checkpoint to write before the update
  if (p.ck_y && n >= p.ck_step0) {
    const unsigned k = (unsigned)(n - p.ck_step0), every = (unsigned)p.ck_every;   // windows hold at most 1e6 steps
    if (k % every == 0 && k / every < p.ck_count) ck = k / every;
  }
  const bool xr = p.xrec && n >= p.xrec_step0 && n - p.xrec_step0 < p.xrec_steps;
#pragma unroll
  for (int c = 0; c < kRounds; ++c) {
    const int jl = tid + c * nthr;
    if (c * nthr < nj && jl < nj) {
      const long long j = j0 + jl;
      long long* slot = p.ring + (size_t)(n & kRingMask) * p.ring_stride + j;
      long long xin = *slot;
      *slot = 0;
      if (ck >= 0) {
        const size_t at = (size_t)ck * p.ring_stride + j;
        p.ck_y[at] = y[c]; p.ck_I[at] = I[c]; p.ck_r[at] = r[c];
      }
      const uint32_t u = quad_drive_word((uint64_t)n, local[c], seed[c]);
      const unsigned pop = (pops[c] >> (8 * (tid & 3))) & 0xFFu;
      if (pop != 0xFFu) {                       // (padding neurons are never updated, never spike)
        xin += (long long)poisson_from_u32(s_table + pop * kTableLen, u) * p.jext_q;
        uint8_t type;
        if (lif_step(p, y[c], I[c], r[c], xin, type)) {
          const int pos = atomicAdd(&s_total, 1);   // in any order: the sums are of integers, the read-back sorts a step
          s_spk[pos] = (int)j;
          s_rs[pos] = rs[c];
          s_len[pos] = (int)(re[c] - rs[c]);
          atomicAdd(&s_events, (unsigned long long)(re[c] - rs[c]));
          atomicAdd(p.wg_spikes + (size_t)blockIdx.x * p.n_pops + pop, 1ull);
        }
        p.y[j] = y[c]; p.I[j] = I[c]; p.r[j] = r[c];
      }
      if (xr) p.xrec[(size_t)(n - p.xrec_step0) * p.ring_stride + j] = xin;
    }
  }
  __syncthreads();
  const int total = s_total;
  if (total == 0) return;

  const bool fits = rbase + total <= p.raster_cap;
  for (int s = tid; s < total && fits; s += nthr)
    p.raster[(size_t)blockIdx.x * p.raster_cap + rbase + s] = make_int2((int)n, s_spk[s]);
  if (tid == 0) {
    if (fits) p.raster_cnt[blockIdx.x] = rbase + total;
    else atomicOr(p.overflow, 1u);
    atomicAdd(p.wg_events + blockIdx.x, s_events);
  }

  if (kOwnerLists) {
    // target-owner scheme: the spikes go to their instance's list of this
    // step; the owner kernel delivers them
    const int par = (int)(n & 1);
    for (int s = tid; s < total; s += nthr) {
      const int i = s_spk[s];
      const int b = p.qinst[i >> 2];
      const int pos = atomicAdd(&p.icnt[par * p.n_inst + b], 1);
      p.ilist[(size_t)par * p.n_pad + p.inst_base[b] + pos] = i;
    }
    return;
  }

  // owner delivery: all threads walk each spiking row in turn, or (wave_rows)
  // every wavefront walks whole rows, the spikes dealt round robin
  const int step = wave_rows ? nthr >> 6 : 1, stride = wave_rows ? 64 : nthr;
  for (int s = wave_rows ? tid >> 6 : 0; s < total; s += step) {
    const long long row = s_rs[s];
    const int len = s_len[s];
    for (int e = wave_rows ? tid & 63 : tid; e < len; e += kAhead * stride) {
      int t[kAhead], w[kAhead], d[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        const int at = e + k * stride;
        if (at < len) { t[k] = p.tgt[row + at]; w[k] = p.wq[row + at]; d[k] = p.dly[row + at]; }
      }
#pragma unroll
      for (int k = 0; k < kAhead; ++k)
        if (e + k * stride < len)
          atomicAdd(reinterpret_cast<unsigned long long*>(p.ring + (size_t)((n + d[k]) & kRingMask) * p.ring_stride + t[k]),
                    (unsigned long long)(long long)w[k]);
    }
  }
}

__global__ void k_advance(long long* step_base, int steps) { *step_base += steps; }

// Adds a value to one ring entry (host-requested input injection).
__global__ void k_inject(long long* ring, long long idx, long long value) { ring[idx] += value; }

// New weights of every synapse in units of 2^-16 pA, rounded to nearest
// even.  kWeightsSet: the real weights w_pA[k]; kWeightsStepF64/F32: one
// gradient step w_q[k] 2^-16 - eta g[k] (g double or float), evaluated as
// fl(w_q 2^-16 - fl(eta g)) (the first product is exact).  check: only test
// that every new weight is finite and fits int32 (*bad = 1 if not), so that a
// rejected update leaves the store untouched; else write them.
enum { kWeightsSet = 0, kWeightsStepF64 = 1, kWeightsStepF32 = 2 };
__global__ void k_weights(int32_t* wq, const void* src, int mode, double eta, long long M, unsigned* bad, int check) {
  for (long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x; k < M; k += (long long)gridDim.x * blockDim.x) {
    double w;
    if (mode == kWeightsSet) {
      w = static_cast<const double*>(src)[k];
    } else {
      const double g = (mode == kWeightsStepF64) ? static_cast<const double*>(src)[k]
                                                 : (double)static_cast<const float*>(src)[k];
      w = (double)wq[k] * 0x1p-16 - eta * g;
    }
    const double ws = w * 65536.0;
    if (check) {
      if (!(fabs(ws) <= 2147483647.0)) atomicOr(bad, 1u);
    } else {
      wq[k] = (int32_t)__double2ll_rn(ws);
    }
  }
}

}  // namespace mc

// ---------------------------------------------------------------------------
// Host-side launch wrappers (called from the C interface)
// ---------------------------------------------------------------------------
namespace mc {

hipError_t launch_step(const DevNet& p, int offset, int qpw, int n_wg, int block, int wave_rows, hipStream_t s) {
  hipLaunchKernelGGL(k_step<false>, dim3(n_wg), dim3(block), 0, s, p, offset, qpw, wave_rows);
  return hipGetLastError();
}

hipError_t launch_step_lists(const DevNet& p, int offset, int qpw, int n_wg, int block, hipStream_t s) {
  hipLaunchKernelGGL(k_step<true>, dim3(n_wg), dim3(block), 0, s, p, offset, qpw, 0);
  return hipGetLastError();
}

hipError_t launch_advance(long long* step_base, int steps, hipStream_t s) {
  hipLaunchKernelGGL(k_advance, dim3(1), dim3(1), 0, s, step_base, steps);
  return hipGetLastError();
}

hipError_t launch_inject(long long* ring, long long idx, long long value, hipStream_t s) {
  hipLaunchKernelGGL(k_inject, dim3(1), dim3(1), 0, s, ring, idx, value);
  return hipGetLastError();
}

hipError_t launch_weights(int32_t* wq, const void* src, int mode, double eta, long long M, unsigned* bad, bool check,
                          hipStream_t s) {
  if (M == 0) return hipSuccess;
  long long blocks = (M + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_weights, dim3((unsigned)blocks), dim3(256), 0, s, wq, src, mode, eta, M, bad, check ? 1 : 0);
  return hipGetLastError();
}

}  // namespace mc
