// mc_persist.hip -- persistent multi-step kernel with the near-future input
// held in LDS (target-owner delivery).
//
// Why: on gfx950 a device-scope int64 atomic is performed at the memory side
// at about 20e9 per second for the whole chip, whatever the footprint of the
// table, so a step of the full microcircuit (~2.5e5 synaptic events) cannot
// drop below ~12 us if every event is a global atomic.  Here every workgroup
// owns a contiguous block of B target neurons (one per thread) and keeps
// their pending input for the next DL steps in LDS (int64, LDS atomics); it
// delivers, for every spike, only the part of the source row that targets its
// own block.  Events with a delay beyond the window (the tail of the delay
// distribution) go to the global ring with device atomics, into entries only
// the owner reads.  The only cross-workgroup traffic per step is the spikes.
//
// Packed rows.  Delivery reads a copy of the store made for this launch shape:
// every row keeps its place (row_ptr) but is reordered by target workgroup,
// the workgroups in XCD order, one 8-byte word per synapse (weight, and the
// delay and local target as one offset into the LDS window), with the sub-row
// bounds of every (row, workgroup) in `off`.
// One load per synapse instead of three, and the 32 workgroups of an XCD read
// adjacent parts of a row, so that cache lines are shared inside one L2.
//
// Wavefront roles.  No barrier runs inside the step loop; the wavefronts of a
// workgroup meet on LDS counters only, so that each part of a step starts as
// soon as its own input is there:
//   - one wavefront (the last) polls the records of step after step and puts
//     the spike ids into a queue in LDS; it may run ahead of the updates;
//   - every wavefront without something more urgent takes ids from the queue
//     and adds all their events (lanes in groups per spike, so that many
//     independent loads are in flight);
//   - a wavefront that owns targets goes through update n as soon as every
//     event of the steps before n is in: input of step n into I, spike
//     decision of step n+1, and the last wavefront to arrive sends the
//     workgroup's record of step n+1.
// With exact integration the spike decision of step m moves y and r with the
// I of before the step; only I <- P11 I + x needs the input read at step m.
// So step n+1's record goes out before step n's records are needed, and the
// exchange (store, visibility, poll) and the delivery overlap over two steps.
//
// Window arithmetic.  Records of step n+1 may be delivered while this
// workgroup's update n has not yet cleared LDS slot n mod DL: an event of
// step n+1 reaches at most slot n+1+d, so only delays d <= DL-2 go to LDS.
// Ids of step n+2 cannot be complete before the own record of step n+1, which
// follows update n, so at most steps n-1..n+2 are in flight and counters by
// step mod 4 suffice.
//
// Spike exchange: workgroup g publishes a record per step (four per
// workgroup, by step mod 4, so a record is never rewritten while a consumer
// may still read it: the record of step n+5 follows update n+4, which needs
// every workgroup's record of step n+3 and hence their delivery of step n+1).
// Word 0 = tag16 << 48 | count << 36 | f with tag16 = (step + 1) mod 65535 + 1
// (never 0, distinct for consecutive steps); up to four spikes, f holds their
// block-local indices (9 bits each), else the mask of the non-zero bitmap
// words L = 1..11, each tag16 << 48 | the spikes of targets 48(L-1)..48L-1.
// About four in five workgroups publish no spike in a step and nearly all
// others at most four, so one load of word 0 usually completes a record.
// Every word carries a tag, so a consumer accepts a record when all the words
// it needs show the current step, whatever order the stores became visible
// in; a tag is the step alone, which suffices because the last workgroup to
// finish a launch clears every record, so that no record outlives the launch
// that wrote it (also across rewinds of the state to earlier steps).  All of
// these are device-scope atomic accesses (coherent at the memory side), so
// the step needs no L2 writeback or invalidate.  Every wait is bounded in
// time (wall clock); on timeout the kernel sets error bit 2 and every
// wavefront leaves its loop.
//
// Bound: latency.  The empty loop of the same exchange takes 1.88 us per step
// (254 workgroups); a quiet step of the full microcircuit 2.6-3.2 us, a burst
// about 19 ns per spike.  Mean over 10,000 steps (barriers, three arrays per
// synapse and a side array of ids -> this form): full microcircuit 9.0 -> 3.9
// us, balanced network 5.0 -> 2.6 us, calls of 20 steps 143-160 -> 86-92 us.
#pragma clang fp contract(off)

#include <algorithm>
#include "mc_device.h"
#include "mc_queue.h"

namespace mc {

namespace {

constexpr int kQueue = 2048;         // spike ids queued in LDS (power of two, >= kPersistMaxB)
constexpr int kW0Ids = 4;            // spike ids in word 0 of a record (9-bit block-local indices)
constexpr int kMapBits = 48;         // targets per bitmap word
constexpr int kMapWords = (kPersistMaxB + kMapBits - 1) / kMapBits;   // 11
// Deliveries (see deliver_few and deliver_many): entries in flight per lane of
// a short claim; units listed per wavefront, and slots of a group in flight, of
// a long one.
constexpr int kFew = 4, kUnits = 64, kSlots = 4;
static_assert(kMapWords <= kWinMapWords, "bitmap words");

// Workgroups are dispatched to the XCDs round robin (workgroup g runs on XCD
// g mod 8), and each XCD has its own L2.  The sub-rows of a source are laid
// out by XCD, so that the parts the workgroups of one XCD read share cache
// lines: position of workgroup g.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_pos(int g, int G) {
  const int x = g % kXcds;
  int pos = g / kXcds;
  for (int y = 0; y < x; ++y) pos += (G - y + kXcds - 1) / kXcds;
  return pos;
}

// Inverse CDF: smallest k with u < T[k] (T ascending, T[63] = 2^32), four
// entries per round of LDS reads.
__device__ __forceinline__ int poisson_inv(const uint64_t* T, uint32_t u) {
  int k = 0;
  for (;;) {
    const ulonglong2 a = *reinterpret_cast<const ulonglong2*>(T + k), b = *reinterpret_cast<const ulonglong2*>(T + k + 2);
    const int c = ((uint64_t)u >= a.x) + ((uint64_t)u >= a.y) + ((uint64_t)u >= b.x) + ((uint64_t)u >= b.y);
    k += c;
    if (c < 4) return k;
  }
}

template <class T>
__device__ __forceinline__ T ld_dev(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void st_dev(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// LDS counters shared by the wavefronts of a workgroup.
template <class T>
__device__ __forceinline__ T lds_acq(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <class T>
__device__ __forceinline__ T lds_rlx(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <class T>
__device__ __forceinline__ void lds_rel(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Inclusive prefix sum over the 64 lanes (row shifts within 16 lanes, then
// the row totals broadcast).
__device__ __forceinline__ int wave_incl(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
  return x;
}

// A value that is the same in every lane, into a scalar register.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ unsigned uni(unsigned x) { return (unsigned)__builtin_amdgcn_readfirstlane((int)x); }
// A wavefront's view of the id queue (see claim_ids): lane k reads the id k
// places on.  The LDS operations of a wavefront are performed in the order in
// which it issues them; the fence keeps the compiler to it and costs nothing.
struct IdQueue {
  const unsigned* slots;
  unsigned mask;                              // slots - 1
  unsigned* s_head;
  int lane;
  unsigned id;
  __device__ __forceinline__ unsigned head() { return uni(lds_rlx(s_head)); }
  __device__ __forceinline__ void read(unsigned h) {
    id = lds_rlx(&slots[(h + (unsigned)lane) & mask]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  __device__ __forceinline__ unsigned take(unsigned h, unsigned to) {
    if (lane == 0)
      __hip_atomic_compare_exchange_strong(s_head, &h, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return uni(h);
  }
};
// Kernel arguments are loaded as tuples of 16 scalar registers, which spill
// and return as a whole; what the step loop uses is copied out one by one,
// the constants of the update into vector registers.
template <class T>
__device__ __forceinline__ T own_s(T x) { asm volatile("" : "+s"(x)); return x; }
// (a pointer comes back as one to global memory: as a generic pointer its
// accesses would be flat ones, which count as LDS accesses too)
template <class T>
__device__ __forceinline__ T* own_p(T* x) {
  typedef __attribute__((address_space(1))) T* global_ptr;
  unsigned long long v = (unsigned long long)x;
  asm volatile("" : "+s"(v));
  return (T*)(global_ptr)v;
}
template <class T>
__device__ __forceinline__ T own_v(T x) { asm volatile("" : "+v"(x)); return x; }

// Poisson counts of the four neurons of a quad at step n, packed in bytes.
__device__ __forceinline__ uint32_t drive_counts(long long n, uint32_t qlocal, uint64_t seed, uint32_t pops,
                                                 const uint64_t* s_table) {
  const U64x4 v = philox4x64_10((uint64_t)n, (uint64_t)qlocal, 0, kTagDrive, seed, 0);
  uint32_t out = 0;
#pragma unroll 1
  for (int k = 0; k < 4; ++k) {               // (not unrolled: the step loop's code has to stay in the instruction cache)
    const unsigned pop = (pops >> (8 * k)) & 0xFFu;
    if (pop == 0xFFu) continue;
    out |= (uint32_t)poisson_inv(s_table + pop * kTableLen, hi32(pick(v, k))) << (8 * k);
  }
  return out;
}

}  // namespace

// LDS (dynamic): acc[DL*B] i64 | fbits[128*BW] u32 | s_q[kQueue] u32 |
//                s_units[kPersistThreads / 64][kUnits] 16 bytes (B is a multiple of 4: all aligned)
// kRec: the adjoint's forward recording (input x and state checkpoints);
// kTime: phase timestamps.  Plain simulation runs the instance with neither
// (fewer registers).  kPoll: producers polled per lane (4 when G <= 256: a
// smaller poll loop, fewer registers; else 8).
template <bool kRec, bool kTime, int kPoll>
__global__ __launch_bounds__(kPersistThreads) void k_persist(DevNet p, PersistArgs a, int steps) {
  extern __shared__ __align__(16) unsigned char s_raw[];
  __shared__ __align__(16) uint64_t s_table[kMaxPops * kTableLen];
  __shared__ uint64_t s_mask[4][kPersistMaxBlock / 64 + 1];   // spike ballots per wavefront, by epoch mod 4 (last: 0)
  __shared__ unsigned long long s_events;
  __shared__ unsigned long long s_popcnt[kMaxPops];
  __shared__ long long s_rcnt;                   // spikes in this workgroup's raster segment
  __shared__ int s_abort, s_last;
  // The id queue: ids [0, s_tail) have been put in, [0, s_head) claimed; of
  // the steps = k (mod 4), s_end[k] ids in listed steps, s_done[k] delivered.
  // s_endq: s_tail after the last step = k (mod 4).
  __shared__ unsigned s_tail, s_head, s_end[4], s_done[4], s_endq[4];
  __shared__ int s_listed;                       // steps of this launch whose records are all in the queue
  __shared__ unsigned s_arr[2];                  // arrivals of the updating wavefronts, by epoch parity (monotonic)
  long long* acc = reinterpret_cast<long long*>(s_raw);
  unsigned* fbits = reinterpret_cast<unsigned*>(acc + (size_t)a.DL * a.B);
  unsigned* s_q = fbits + 128 * a.BW;
  uint4* s_units = reinterpret_cast<uint4*>(s_q + kQueue);          // [wavefronts][kUnits] 

  const int g = blockIdx.x, tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, nw = nthr >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gpos = xcd_pos(g, a.G);                                 // place of this workgroup in a packed row
  const long long j0 = a.bstart[g];                                 // first owned target (padded id)
  const int Bg = a.bstart[g + 1] - a.bstart[g];                     // owned targets (multiple of 4, <= B)
  const long long n0 = *p.step_base;
  const int DL = own_s(a.DL), B = own_s(a.B), BW = own_s(a.BW), G = own_s(a.G);
  long long* const ring = own_p(p.ring) + j0;                       // my targets' entries of slot 0
  const unsigned ring_stride = own_s((unsigned)p.ring_stride);
  unsigned long long* const flags = own_p(a.flags);
  const double P11 = own_v(p.P11), P21 = own_v(p.P21), P22 = own_v(p.P22), theta = own_v(p.theta), y_reset = own_v(p.y_reset);
  const double drift = own_v(p.P20 * p.i_e);
  const bool drifts = p.i_e != 0.0;
  const long long jext_q = own_v(p.jext_q);
  const int ref_steps = own_v(p.ref_steps);
  // the queue's capacity and slots (a test hook makes them fewer, in the
  // phase-timing instance only; what the poller puts in at once always fits:
  // the ids of a long record, or of the short records that a lane polls)
  unsigned qcap = kQueue, qmask = kQueue - 1;
  if (kTime && a.list_cap > 0) {
    qcap = (unsigned)min(max(a.list_cap, max(B, kW0Ids * kPoll)), kQueue);
    qmask = (1u << (32 - __builtin_clz(qcap - 1))) - 1;
  }

  for (int k = tid; k < p.n_pops * kTableLen; k += nthr) s_table[k] = p.table[k];
  for (int k = tid; k < DL * B; k += nthr) acc[k] = 0;
  for (int k = tid; k < 128 * a.BW; k += nthr) fbits[k] = 0;
  if (tid < 4 * (kPersistMaxBlock / 64 + 1)) (&s_mask[0][0])[tid] = 0;
  if (tid < 4) { s_end[tid] = 0; s_done[tid] = 0; }
  if (tid == 0) { s_abort = 0; s_events = 0; s_tail = 0; s_head = 0; s_listed = 0; s_arr[0] = 0; s_arr[1] = 0; s_rcnt = p.raster_cnt[g]; }
  if (tid < kMaxPops) s_popcnt[tid] = 0;
  __syncthreads();

  // ---- roles ------------------------------------------------------------------
  const int nupd = (Bg + 63) >> 6;                 // wavefronts that own targets
  const bool isU = wave < nupd;
  const bool isP = wave == nw - 1;                 // the poller
  // A poller that is also the workgroup's only wavefront delivers as well;
  // otherwise the poller leaves the queue to the others.
  const bool delivers = !isP || nw == 1;

  // neuron state in registers: thread t < Bg owns neuron j0+t
  double y = 0.0, I = 0.0;
  int r = 0;
  unsigned pop = 0xFFu;
  uint32_t qlocal = 0, qpops = 0xFFFFFFFFu;
  uint64_t seed = 0;
  const bool upd = tid < Bg;
  const int qk = tid & 3;
  // Drive: one Philox block gives the four neurons of a quad at one step, so
  // the four threads of a quad draw four consecutive steps (one each) and
  // pass each other their counts: a block per thread every four steps.
  uint32_t kpack = 0;
  int kdrive = 0;
  if (upd) {
    const long long q = (j0 + tid) >> 2;
    qpops = p.qpops[q]; qlocal = p.qlocal[q]; seed = p.qseed[q];
    pop = (qpops >> (8 * qk)) & 0xFFu;
    y = p.y[j0 + tid]; I = p.I[j0 + tid]; r = p.r[j0 + tid];
    kpack = drive_counts(n0 + qk, qlocal, seed, qpops, s_table);
  }
  auto drive_of = [&](int idx) -> int {            // my neuron's count at step idx of the four drawn
    return (int)((__shfl(kpack, (lane & ~3) | idx, 64) >> (8 * qk)) & 0xFFu);
  };
  if (isU) kdrive = drive_of(0);
  // checkpoint schedule of an adjoint's forward: segment of step n0 and n0's
  // phase in it (a checkpoint is due at phase 0)
  long long ck_seg = -1, ck_phase = 1;
  if (kRec && p.ck_y) {
    const long long k = n0 - p.ck_step0;
    ck_seg = (k >= 0) ? k / p.ck_every : -1;
    ck_phase = (k >= 0) ? k % p.ck_every : 1;
  }
  long long ph[7] = {0, 0, 0, 0, 0, 0, 0};

  auto decide = [&](long long m) -> int {     // spike decision of step m
    if (kRec && p.ck_y) {                   // adjoint forward: checkpoint before the update
      if (upd && ck_phase == 0 && ck_seg >= 0 && ck_seg < p.ck_count) {
        const size_t at = (size_t)ck_seg * p.ring_stride + j0 + tid;
        p.ck_y[at] = y; p.ck_I[at] = I; p.ck_r[at] = r;
      }
      if (++ck_phase == p.ck_every) { ck_phase = 0; ++ck_seg; }
    }
    int spiked = 0;
    if (upd && pop != 0xFFu) {
      const bool free_ = (r == 0);
      if (free_) {
        double yn = P22 * y + P21 * I;
        if (drifts) yn = yn + drift;
        y = yn;
      } else {
        r = r - 1;
      }
      if (free_ && y >= theta) {
        y = y_reset;
        r = ref_steps;
        spiked = 1;
        atomicAdd(&s_popcnt[pop], 1ull);
      }
    }
    return spiked;
  };
  auto absorb = [&](long long m, int slot) {  // input of step m into I; its LDS slot cleared
    if (!upd) return;
    const int fslot = (int)(m & kRingMask);
    const int jl = tid;
    long long x_int = acc[slot * B + jl];
    acc[slot * B + jl] = 0;
    unsigned* fb = &fbits[fslot * BW + (jl >> 5)];
    if (*fb & (1u << (jl & 31))) {
      atomicAnd(fb, ~(1u << (jl & 31)));
      x_int += (long long)__hip_atomic_exchange(
          reinterpret_cast<unsigned long long*>(ring + (size_t)fslot * ring_stride + jl), 0ull,
          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (pop != 0xFFu) x_int += (long long)kdrive * jext_q;
    if (kRec && p.xrec && m - p.xrec_step0 >= 0 && m - p.xrec_step0 < p.xrec_steps)
      p.xrec[(size_t)(m - p.xrec_step0) * p.ring_stride + j0 + jl] = x_int;
    if (pop != 0xFFu) I = P11 * I + (double)x_int * 0x1p-16;
  };
  // Compaction (thread order = id order): the ballots of the updating
  // wavefronts meet in LDS; the wavefront that arrives last sends the record
  // of step m, then appends the spikes to the raster.
  // t16m = (m + 1) mod 65535 + 1; epoch = m - n0.  A fast wavefront may arrive
  // for epoch e+1 before a slow one has for e, but not for e+2: its update
  // then needs this workgroup's record of epoch e.  So arrivals are counted
  // by epoch parity; the ballots of epoch e are overwritten at e+4, when the
  // wavefront that arrived last for e has arrived for e+2.
  auto publish = [&](long long m, int spiked, unsigned t16m, int epoch) {
    const int buf = epoch & 3;
    const uint64_t bal = __ballot(spiked);
    int last = 0;
    if (lane == 0) {
      s_mask[buf][wave] = bal;
      last = (__hip_atomic_fetch_add(&s_arr[epoch & 1], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) + 1u ==
              (unsigned)nupd * (unsigned)((epoch >> 1) + 1));
    }
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const uint64_t* msk = s_mask[buf];
    const unsigned long long tag = (unsigned long long)t16m << 48;
    uint64_t mr[kPersistMaxBlock / 64];         // all masks, loaded together
#pragma unroll
    for (int w = 0; w < kPersistMaxBlock / 64; ++w) mr[w] = msk[w];   // (zero beyond nupd)
    const int mapw = (kMapBits * lane) >> 6, sh = (kMapBits * lane) & 63;   // lane L < 11 holds targets 48L..48L+47
    const uint64_t m_lo = msk[min(mapw, kPersistMaxBlock / 64)], m_hi = msk[min(mapw + 1, kPersistMaxBlock / 64)];
    int nloc = 0;
#pragma unroll
    for (int w = 0; w < kPersistMaxBlock / 64; ++w) nloc += __popcll(mr[w]);
    nloc = uni(nloc);
    unsigned long long f = 0;
    if (nloc > kW0Ids) {
      unsigned long long v = m_lo >> sh;
      if (sh > 64 - kMapBits) v |= m_hi << (64 - sh);
      v &= (1ull << kMapBits) - 1;
      if (lane >= kMapWords) v = 0;
      f = __ballot(v != 0);
      if (v != 0) st_dev(&flags[window_map(G, (int)(m & (kRecSlots - 1)), g) + lane], tag | v);
    } else if (nloc > 0) {
      int k = 0;
#pragma unroll
      for (int w = 0; w < kPersistMaxBlock / 64; ++w)
        for (uint64_t mm = mr[w]; mm; mm &= mm - 1, ++k) f |= (unsigned long long)(64 * w + __builtin_ctzll(mm)) << (9 * k);
    }
    if (lane == 0) st_dev(&flags[window_word0(G, (int)(m & (kRecSlots - 1)), g)], tag | (unsigned long long)nloc << 36 | f);
    if (nloc == 0) return;
    const long long rcnt = s_rcnt;
    if (rcnt + nloc <= p.raster_cap) {
      int2* out = p.raster + (size_t)g * p.raster_cap + rcnt;
#pragma unroll
      for (int w = 0; w < kPersistMaxBlock / 64; ++w) {
        const uint64_t mm = mr[w];
        if ((mm >> lane) & 1ull)
          out[__popcll(mm & (lane ? (~0ull >> (64 - lane)) : 0ull))] = make_int2((int)m, (int)(j0 + 64 * w + lane));
        out += __popcll(mm);
      }
      if (lane == 0) s_rcnt = rcnt + nloc;
    } else if (lane == 0) {
      atomicOr(p.overflow, 1u);
    }
  };

  static_assert((kRecSlots & (kRecSlots - 1)) == 0, "record slots by step & (kRecSlots - 1)");
  auto next16 = [](unsigned t) { return t == 65535u ? 1u : t + 1u; };
  const unsigned t16_0 = (unsigned)((n0 + 1) % 65535 + 1);   // tag of step n0's record
  unsigned t16u = t16_0;                      // tag of the record sent last (advanced with every update)
  if (steps > 0 && isU) {                     // step n0's spike decision and record
    const int sp = decide(n0);
    publish(n0, sp, t16u, 0);
  }
  // Then take the next DL steps of pending input of my targets into LDS and
  // mark far entries (step n0's decision does not need them, so every
  // workgroup's first record is out while this scan runs).  Only the first
  // `horizon` slots can hold input (the largest delay, or further after an
  // injection or a loaded state).  Inside a launch only the owner workgroup
  // touches its targets' ring entries, so device-scope loads and stores
  // suffice (no read-modify-write).  A wavefront takes whole slots, eight at
  // a time, so that all slot arithmetic is scalar and eight loads per lane
  // are in flight.
  {
    const int take = min(DL, a.horizon), scan = min(127, a.horizon);
    const int sl0 = (int)(n0 % DL), rs0 = (int)(n0 & kRingMask);   // LDS and ring slot of step n0
    constexpr int kPro = 8;
    for (int m0 = wave; m0 < scan; m0 += kPro * nw) {
      for (int jl = lane; jl < Bg; jl += 64) {
        long long v[kPro];
#pragma unroll
        for (int u = 0; u < kPro; ++u) {
          const int m = m0 + u * nw;
          v[u] = (m < scan) ? ld_dev(ring + (size_t)((rs0 + m) & kRingMask) * ring_stride + jl) : 0ll;
        }
#pragma unroll
        for (int u = 0; u < kPro; ++u) {
          const int m = m0 + u * nw, rs = (rs0 + m) & kRingMask;
          if (v[u] == 0) continue;
          if (m < take) {
            const int s = sl0 + m;
            acc[(s >= DL ? s - DL : s) * B + jl] = v[u];
            st_dev(ring + (size_t)rs * ring_stride + jl, 0ll);
          } else if (m >= DL) {
            atomicOr(&fbits[rs * BW + (jl >> 5)], 1u << (jl & 31));
          }
        }
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();                            // the window is in LDS before step n0's input is read

  // ---- step loop of a wavefront ------------------------------------------------
  const int ls = a.lsh;                       // lanes per id of a delivery: 1 << ls
  const int sub = lane >> ls, sl_lane = lane & ((1 << ls) - 1), per = 64 >> ls;
  const unsigned* const off = own_p(a.off) + gpos;   // sub-row bounds of this workgroup in row 0
  const unsigned long long* const pk = own_p(a.pk);
  const int64_t* const row_ptr = own_p(p.row_ptr);
  const long long wait_ticks = own_s(a.wait_ticks);
  unsigned long long ev = 0;                  // synaptic events delivered by this lane's sub-rows
  int uit = 0, un = (int)(n0 % DL);           // next update (step n0 + uit) and its LDS slot
  int pit = 0, pn = (int)(n0 % DL);           // the poller's step and its LDS slot
  unsigned t16p = t16_0, tail = 0;            // its tag; ids put into the queue
  unsigned todo = 0, todo_all = 0;            // producers of the step still to be seen
  if (isP) {
#pragma unroll
    for (int k = 0; k < kPoll; ++k)
      if (lane + 64 * k < G) todo_all |= 1u << k;
    todo = todo_all;
  }
  const unsigned B8 = (unsigned)B * 8u, win = own_s((unsigned)DL * B8);   // bytes of a slot and of the window
  const unsigned near_span = (unsigned)(DL - 2) * B8;    // offsets B8 .. B8 + near_span - 1: delays 1 .. DL-2
  unsigned char* const acc_b = reinterpret_cast<unsigned char*>(acc);
  // One event: packed entry e of a spike whose slot starts at byte sn of the
  // window (entry 0 or sn kNone: the lane has none here).
  // Returns whether it lies beyond the window (add_far).
  constexpr unsigned kNone = 0x80000000u;
  auto add = [&](unsigned long long e, unsigned sn) __attribute__((always_inline)) -> bool {
    const unsigned hi = (int)sn < 0 ? 0u : (unsigned)(e >> 32), at = sn + hi;
    if (hi - B8 < near_span)
      atomicAdd(reinterpret_cast<unsigned long long*>(acc_b + min(at, at - win)),   // modulo the window
                (unsigned long long)(long long)(int)(e & 0xFFFFFFFFu));
    return hi >= B8 + near_span;
  };
  auto add_far = [&](unsigned long long e, unsigned rs) {   // rs: the spike's ring slot
    const unsigned hi = (unsigned)(e >> 32);
    const unsigned d = hi / B8, jl = (hi - d * B8) >> 3, fs = (rs + d) & (unsigned)kRingMask;
    atomicAdd(reinterpret_cast<unsigned long long*>(ring + (size_t)fs * ring_stride + jl),
              (unsigned long long)(long long)(int)(e & 0xFFFFFFFFu));
    atomicOr(&fbits[fs * BW + (jl >> 5)], 1u << (jl & 31));
  };
  // The claim's ids (one per lane in qq) are delivered.  far: some event went
  // to the ring, whose add must be complete first.  A claim may span steps.
  auto delivered = [&](unsigned qq, unsigned c, bool far) {
    if (far) __builtin_amdgcn_s_waitcnt(0);
    for (unsigned long long rem = c >= 64 ? ~0ull : (1ull << c) - 1; rem;) {
      const unsigned st = (unsigned)__builtin_amdgcn_readlane((int)qq, __builtin_ctzll(rem)) >> 25 & 3u;
      const unsigned long long same = __ballot((qq >> 25 & 3u) == st) & rem;
      rem &= ~same;
      if (lane == 0)
        __hip_atomic_fetch_add(&s_done[st], (unsigned)__popcll(same), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  };
  // All events of the c claimed ids (lane k holds id k in qq; lanes >= c
  // unused), c <= per: a group of 1 << ls lanes per id, kFew entries in flight
  // per lane.  The fewest instructions for the few spikes of a quiet step.
  auto deliver_few = [&](unsigned qq, unsigned c) {
    const unsigned q = (unsigned)__shfl((int)qq, sub, 64);
    const bool mine = sub < (int)c;
    const unsigned id = mine ? q & 0x3FFFFu : 0u;
    const unsigned* o = off + (size_t)id * (unsigned)(G + 1);
    const long long rp = row_ptr[id];
    const unsigned o0 = o[0], o1 = o[1];
    __builtin_amdgcn_sched_barrier(0);                      // all three loads are out before the first is waited for
    const long long ent = rp + o0 + sl_lane;
    int len = mine ? (int)(o1 - o0) : 0;
    const unsigned sn = __umul24((q >> 18) & 0x7Fu, B8);
    if (sl_lane == 0) ev += (unsigned)len;
    len -= sl_lane;                                         // this lane's entries: 0, L, 2L, ... < len
    bool far = false;
    for (int e = 0; __any(e < len); e += kFew << ls) {
      unsigned long long v[kFew];
      bool beyond = false;
#pragma unroll
      for (int u = 0; u < kFew; ++u) {
        const bool ok = e + (u << ls) < len;
        v[u] = 0;
        if (ok) v[u] = pk[ent + e + (u << ls)];
      }
#pragma unroll
      for (int u = 0; u < kFew; ++u) beyond |= add(v[u], sn);
      if (__any(beyond)) {                                  // rare
        far = true;
#pragma unroll
        for (int u = 0; u < kFew; ++u)
          if ((unsigned)(v[u] >> 32) >= B8 + near_span) add_far(v[u], q >> 25);
      }
    }
    delivered(qq, c, far);
  };
  // All events of the c claimed ids, c <= 64: a lane per id finds its sub-row and
  // cuts it into units of 1 << ls entries, listed in LDS; then the wavefront
  // walks the units, 64 / L at a time (a slot), two groups of kSlots slots in
  // flight.  One chain of dependent loads per claim and few idle lanes: the
  // full microcircuit's bursts (600 to 3,000 spikes a step) went from 35 to 22 ns
  // per spike with the units and to 19 with 12 wavefronts instead of 8.
  auto deliver_many = [&](unsigned qq, unsigned c) {
    const bool mine = lane < (int)c;
    const unsigned id = mine ? qq & 0x3FFFFu : 0u;
    const unsigned* o = off + (size_t)id * (unsigned)(G + 1);
    const long long rp = row_ptr[id];
    const unsigned o0 = o[0], o1 = o[1];
    __builtin_amdgcn_sched_barrier(0);
    const long long first = rp + o0;
    const int len = mine ? (int)(o1 - o0) : 0;
    ev += (unsigned)len;
    const unsigned sn = __umul24((qq >> 18) & 0x7Fu, B8);
    const int units = (len + (1 << ls) - 1) >> ls;
    const int x = wave_incl(units), total = __builtin_amdgcn_readlane(x, 63), base = x - units;
    uint4* const ul = s_units + wave * kUnits;              // this wavefront's
    bool far = false;
    for (int w0 = 0; w0 < total; w0 += kUnits) {
      const int je = min(units, w0 + kUnits - base);
      for (int j = max(0, w0 - base); j < je; ++j) {
        const long long at = first + (j << ls);
        ul[base + j - w0] = make_uint4((unsigned)at, (unsigned)(at >> 32), (unsigned)min(1 << ls, len - (j << ls)) | (qq >> 25) << 16, sn);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int nu = min(kUnits, total - w0);
      const int groups = (nu + kSlots * per - 1) / (kSlots * per);
      unsigned long long va[kSlots], vb[kSlots];
      unsigned na[kSlots], nb[kSlots];
      // (every lane loads, from a safe address if it has no entry, so that the
      // wait for one group in flight leaves the other alone)
      auto load = [&](unsigned long long* v, unsigned* sb, int grp) __attribute__((always_inline)) {
        uint4 t[kSlots];
        const int i0 = grp * kSlots * per + sub;
#pragma unroll
        for (int u = 0; u < kSlots; ++u) t[u] = ul[min(i0 + u * per, kUnits - 1)];
#pragma unroll
        for (int u = 0; u < kSlots; ++u) {
          const bool ok = i0 + u * per < nu && sl_lane < (int)(t[u].z & 0xFFFFu);
          v[u] = pk[ok ? (long long)((unsigned long long)t[u].y << 32 | t[u].x) + sl_lane : 0ll];
          sb[u] = ok ? t[u].w : kNone;
        }
      };
      auto process = [&](const unsigned long long* v, const unsigned* sb, int grp) __attribute__((always_inline)) {
        bool beyond = false;
#pragma unroll
        for (int u = 0; u < kSlots; ++u) beyond |= add(v[u], sb[u]);
        if (__any(beyond)) {                                // rare
          far = true;
#pragma unroll
          for (int u = 0; u < kSlots; ++u)
            if ((int)sb[u] >= 0 && (unsigned)(v[u] >> 32) >= B8 + near_span)
              add_far(v[u], ul[(grp * kSlots + u) * per + sub].z >> 16);
        }
      };
      load(va, na, 0);
      for (int grp = 0; grp < groups; grp += 2) {
        if (grp + 1 < groups) load(vb, nb, grp + 1);
        process(va, na, grp);
        if (grp + 2 < groups) load(va, na, grp + 2);
        if (grp + 1 < groups) process(vb, nb, grp + 1);
      }
      __builtin_amdgcn_wave_barrier();
    }
    delivered(qq, c, far);
  };
  unsigned spins = 0;
  long long t_wait = 0;                       // wall clock at the first check of a wait (0: not waiting)
  long long tp_idle = kTime ? wall_clock64() : 0;

  // The poller and the updates are the step's critical path: they issue ahead
  // of the wavefronts that deliver (full microcircuit 4.27 -> 3.98 us per step,
  // balanced 2.89 -> 2.58).
  if (isP) __builtin_amdgcn_s_setprio(3);
  for (;;) {
    // ---- update: input of step n into I, spike decision and record of step
    //      n+1, once every event of the steps before n is in ---------------------
    bool limited = false;                     // claim only ids before limit (but see below)
    unsigned limit = 0;
    if (isU && uit < steps) {
      const long long n = n0 + uit;
      bool ready = uit == 0;
      if (!ready && uni(lds_acq(&s_listed)) >= uit) {
        const int k = (int)((n - 1) & 3);
        limited = true;
        limit = uni(s_endq[k]);
        ready = uni(lds_acq(&s_done[k]) - s_end[k]) == 0;
      }
      if (ready) {
        __builtin_amdgcn_s_setprio(3);
        long long tp = 0;
        if (kTime) { tp = wall_clock64(); ph[2] += tp - tp_idle; }
        absorb(n, un);
        int spiked = 0;
        const bool more = uit + 1 < steps;
        if (more) spiked = decide(n + 1);
        if (kTime) { const long long t = wall_clock64(); ph[0] += t - tp; tp = t; }
        t16u = next16(t16u);
        if (more) publish(n + 1, spiked, t16u, uit + 1);
        if (kTime) { const long long t = wall_clock64(); ph[1] += t - tp; tp = t; }
        un = (un + 1 == DL) ? 0 : un + 1;
        ++uit;
        if (more) {
          if ((uit & 3) == 0 && upd) kpack = drive_counts(n + 1 + qk, qlocal, seed, qpops, s_table);
          kdrive = drive_of(uit & 3);
        }
        if (kTime) { tp_idle = wall_clock64(); ph[5] += tp_idle - tp; }
        t_wait = 0;
        if (!isP) __builtin_amdgcn_s_setprio(0);
        continue;
      }
    }
    bool progress = false;
    // ---- poll: the records of step n0 + pit; their ids into the queue ---------
    // (an updating poller first sends its own workgroup's record of that step)
    if (isP && pit < steps && (!isU || pit <= uit)) {
      const long long tq = kTime ? wall_clock64() : 0;
      const long long n = n0 + pit;
      const int rslot = (int)(n & (kRecSlots - 1));
      const unsigned long long* recs = flags + window_word0(G, rslot, 0);
      const unsigned qtag = (unsigned)pn << 18 | (unsigned)(n & kRingMask) << 25;
      const unsigned tail0 = tail;
      unsigned long long w0[kPoll];
#pragma unroll
      for (int k = 0; k < kPoll; ++k) w0[k] = ((todo >> k) & 1u) ? ld_dev(&recs[(lane + 64 * k) * kWord0Stride]) : 0ull;
      const unsigned gone = lds_rlx(&s_done[0]) + lds_rlx(&s_done[1]) + lds_rlx(&s_done[2]) + lds_rlx(&s_done[3]);   // ids delivered by now (the queue's room)
      // records of up to four spikes: their ids are in word 0
      unsigned few = 0, many = 0, cf = 0;       // the k of this lane's records by size; ids of the short ones
#pragma unroll
      for (int k = 0; k < kPoll; ++k) {
        const unsigned hi = (unsigned)(w0[k] >> 32), c = (hi >> 4) & 0xFFFu;
        if (((todo >> k) & 1u) && (hi >> 16) == t16p) {
          if (c <= (unsigned)kW0Ids) { few |= 1u << k; cf += c; }
          else many |= 1u << k;
        }
      }
      if (!__any(cf != 0)) {
        todo &= ~few;                           // nothing but empty records
      } else {
        const int x = wave_incl((int)cf);
        const bool ok = x <= (int)queue_room(qcap, tail, gone);   // room in the queue: the accepted lanes are a prefix
        if (ok) {
          todo &= ~few;
          unsigned o = tail + (unsigned)x - cf;
#pragma unroll
          for (int k = 0; k < kPoll; ++k) {
            const unsigned c = ((few >> k) & 1u) ? ((unsigned)(w0[k] >> 36) & 0xFFFu) : 0u;
            const unsigned b = (unsigned)((lane + 64 * k) * B) | qtag;   // ids < 2^18, with a local index too: no carry
#pragma unroll
            for (int e = 0; e < kW0Ids; ++e)
              if ((unsigned)e < c) s_q[(o + (unsigned)e) & qmask] = b + ((unsigned)(w0[k] >> (9 * e)) & 0x1FFu);
            o += c;
          }
        }
        const unsigned long long acc_m = __ballot(ok);
        if (acc_m) tail += (unsigned)__builtin_amdgcn_readlane(x, 63 - __builtin_clzll(acc_m));
        if (lane == 0) lds_rel(&s_tail, tail);
      }
      // longer records: 16 lanes read the bitmap words of one, sixteen records
      // in flight; a lane puts in the ids of its word
      if (__any(many != 0)) {
#pragma unroll 1
        for (int k = 0; k < kPoll; ++k) {
          unsigned long long w = w0[0];
#pragma unroll
          for (int u = 1; u < kPoll; ++u) w = (u == k) ? w0[u] : w;
          unsigned long long left = __ballot((many >> k) & 1u);
          const int L = lane & 15, rr = lane >> 4;
          while (left) {
            constexpr int kBatch = 4;
            unsigned long long wk[kBatch];
            int own[kBatch];                    // the lane that polls this group's record (-1: none)
            bool need[kBatch];
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
              own[q] = -1;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int l = left ? __builtin_ctzll(left) : -1;
                left &= left - 1;               // (0 stays 0)
                own[q] = (rr == e) ? l : own[q];
              }
              const unsigned long long wr = __shfl(w, own[q] & 63, 64);
              need[q] = own[q] >= 0 && L < kMapWords && ((wr >> L) & 1ull);
              wk[q] = 0;
              if (need[q]) wk[q] = ld_dev(&flags[window_map(G, rslot, own[q] + 64 * k) + L]);
            }
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
              const unsigned long long bad = __ballot(need[q] && (unsigned)(wk[q] >> 48) != t16p);
              const bool good = own[q] >= 0 && ((bad >> (lane & 48)) & 0xFFFFull) == 0;
              unsigned long long mm = (good && need[q]) ? wk[q] & ((1ull << kMapBits) - 1) : 0ull;
              const int x = wave_incl(__popcll(mm)), xr = __shfl(x, lane | 15, 64);   // up to the end of the record
              const bool ok = good && xr <= (int)queue_room(qcap, tail, gone);
              if (ok) {
                unsigned o = tail + (unsigned)(x - __popcll(mm));
                const unsigned b = ((unsigned)((own[q] + 64 * k) * B) | qtag) + (unsigned)(kMapBits * L);
                for (; mm; mm &= mm - 1) s_q[o++ & qmask] = b + (unsigned)__builtin_ctzll(mm);
              }
              const unsigned long long acc_m = __ballot(ok);
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if ((acc_m >> (16 * e)) & 1ull && lane == __builtin_amdgcn_readlane(own[q], 16 * e)) todo &= ~(1u << k);
              if (acc_m) tail += (unsigned)__builtin_amdgcn_readlane(x, 63 - __builtin_clzll(acc_m));
            }
            if (lane == 0) lds_rel(&s_tail, tail);
          }
        }
      }
      progress = tail != tail0;
      const bool complete = !__any(todo != 0);
      if (complete) {
        if (lane == 0) {
          const int k = (int)(n & 3);
          // the ids of this step: all put in so far less those of the other steps
          s_end[k] = tail - s_end[(k + 1) & 3] - s_end[(k + 2) & 3] - s_end[(k + 3) & 3];
          s_endq[k] = tail;
          lds_rel(&s_listed, pit + 1);
        }
        progress = true;
        todo = todo_all;
        ++pit;
        t16p = next16(t16p);
        pn = (pn + 1 == DL) ? 0 : pn + 1;
      }
      if (kTime) ph[6] += wall_clock64() - tq;
    }
    // ---- deliver: claim ids and add all their events ---------------------------
    if (delivers || (pit == steps && uit >= (isU ? steps : 0))) {
      unsigned t = uni(lds_acq(&s_tail));
      // later steps' ids are not what an update waits for: it leaves them to
      // the other wavefronts unless many pile up (a burst)
      if (limited && (int)(t - limit) <= nw * per) t = limit;
      IdQueue queue{s_q, qmask, &s_head, lane, 0u};
      const unsigned c = claim_ids(queue, t, (unsigned)per, (unsigned)nw);
      if (c > 0) {
        const long long tq = kTime ? wall_clock64() : 0;
        if (c <= (unsigned)per) deliver_few(queue.id, c);
        else deliver_many(queue.id, c);
        if (kTime) { const long long t = wall_clock64(); ph[4] += t - tq; tp_idle += t - tq; }
        t_wait = 0;
        continue;
      }
    }
    if (progress) { t_wait = 0; continue; }
    // ---- nothing to do now -------------------------------------------------------
    if ((!isU || uit == steps) && (!isP || pit == steps) && uni(lds_acq(&s_listed)) == steps &&
        uni(lds_rlx(&s_head) - lds_rlx(&s_tail)) == 0)
      break;
    if (uni(lds_rlx(&s_abort))) break;
    if (!isU) __builtin_amdgcn_s_sleep(1);
    // (a wavefront that only delivers may rightly idle for long)
    if ((isP || isU) && (++spins & 255u) == 0u) {   // the wall clock is read every 256 rounds only
      const long long t = wall_clock64();
      if (t_wait == 0) t_wait = t;
      else if (t - t_wait > wait_ticks) {
        if (lane == 0) atomicOr(p.overflow, 2u);
        s_abort = 1;
        break;
      }
    }
  }
  const long long n_end = n0 + steps;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ev += __shfl_xor(ev, o, 64);
  if (lane == 0 && ev) atomicAdd(&s_events, ev);
  __syncthreads();
  // ---- epilogue: state, counters, LDS window back into the global ring ------
  if (upd) { p.y[j0 + tid] = y; p.I[j0 + tid] = I; p.r[j0 + tid] = r; }
  if (tid < p.n_pops) p.wg_spikes[(size_t)g * p.n_pops + tid] += s_popcnt[tid];
  if (kTime && tid == 0) {
    for (int k = 0; k < 6; ++k) a.phase[(size_t)g * 8 + k] += (unsigned long long)ph[k];
    a.phase[(size_t)g * 8 + 7] += (unsigned long long)steps;
  }
  if (kTime && tid == nthr - 64) a.phase[(size_t)g * 8 + 6] += (unsigned long long)ph[6];
  if (tid == 0) {
    p.raster_cnt[g] = s_rcnt;
    p.wg_events[g] += s_events;
  }
  // the global entry of a window slot is zero unless far events were added
  // to it (its far bit): a store, else an add
  {
    const int sl0 = (int)(n_end % DL), rs0 = (int)(n_end & kRingMask);
    for (int m = wave; m < DL; m += nw) {
      const int s = (sl0 + m >= DL) ? sl0 + m - DL : sl0 + m, rs = (rs0 + m) & kRingMask;
      for (int jl = lane; jl < Bg; jl += 64) {
        const long long v = acc[s * B + jl];
        if (v == 0) continue;
        long long* e = ring + (size_t)rs * ring_stride + jl;
        if (fbits[rs * BW + (jl >> 5)] & (1u << (jl & 31)))
          atomicAdd(reinterpret_cast<unsigned long long*>(e), (unsigned long long)v);
        else
          st_dev(e, v);
      }
    }
  }
  // The last workgroup to finish (every other one has read all the records it
  // will read) clears the spike records for the next launch and advances the
  // step counter (every workgroup read it before its first record).
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (tid == 0) {
    unsigned long long* done = a.flags + window_record_words(a.G);
    s_last = (__hip_atomic_fetch_add(done, 1ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (unsigned long long)(a.G - 1));
  }
  __syncthreads();
  if (s_last) {
    const int words = (int)window_record_words(a.G);
    for (int k = tid; k < words; k += nthr) st_dev(&a.flags[k], 0ull);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
      st_dev(p.step_base, n_end);
      __hip_atomic_store(a.flags + window_record_words(a.G), 0ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// The exchange of k_persist with nothing else: every step, each of the G
// workgroups publishes a step-tagged record (word 0 as in k_persist, no
// spikes) and its last wavefront polls all G records of the step the same
// way (four or eight producers per lane, device-scope loads, a short sleep between
// rounds); then a barrier and the next step.  The time per step is the floor
// the persistent kernel's step cannot go below.  Records are cleared by the
// last workgroup to finish, as in k_persist.
template <int kPoll>
__global__ __launch_bounds__(kPersistMaxBlock) void k_exchange_probe(unsigned long long* flags, int G, long long steps,
                                                                     long long wait_ticks, unsigned* err) {
  __shared__ int s_abort, s_last;
  const int g = blockIdx.x, tid = threadIdx.x, nthr = blockDim.x;
  const int nw = nthr >> 6, wave = tid >> 6, lane = tid & 63;
  if (tid == 0) s_abort = 0;
  __syncthreads();
  for (long long n = 0; n < steps; ++n) {
    const unsigned long long tag16 = (unsigned long long)((n + 1) % 65535 + 1) << 48;
    const size_t rslot = (size_t)(n % kRecSlots);
    if (tid == 0) st_dev(&flags[window_word0(G, (int)rslot, g)], tag16);
    if (wave == nw - 1) {
      long long t_poll = 0;          // the wall clock is read every 256 rounds only
      unsigned spins = 0;
      unsigned todo = 0;
#pragma unroll
      for (int r = 0; r < kPoll; ++r)
        if (lane + 64 * r < G) todo |= 1u << r;
      while (todo) {
        unsigned long long w0[kPoll];
#pragma unroll
        for (int r = 0; r < kPoll; ++r)
          w0[r] = ((todo >> r) & 1u) ? ld_dev(&flags[window_word0(G, (int)rslot, lane + 64 * r)])
                                     : 0ull;
#pragma unroll
        for (int r = 0; r < kPoll; ++r)
          if (((todo >> r) & 1u) && (w0[r] & 0xFFFF000000000000ull) == tag16) todo &= ~(1u << r);
        if (!todo) break;
        __builtin_amdgcn_s_sleep(1);
        if ((++spins & 255u) == 0u && (t_poll == 0 ? ((t_poll = wall_clock64()), false) : wall_clock64() - t_poll > wait_ticks)) {
          atomicOr(err, 2u);
          s_abort = 1;
          break;
        }
      }
    }
    __syncthreads();
    if (s_abort) break;
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (tid == 0) {
    unsigned long long* done = flags + window_record_words(G);
    s_last = (__hip_atomic_fetch_add(done, 1ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (unsigned long long)(G - 1));
  }
  __syncthreads();
  if (s_last) {
    const int words = (int)window_record_words(G);
    for (int k = tid; k < words; k += nthr) st_dev(&flags[k], 0ull);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) __hip_atomic_store(flags + window_record_words(G), 0ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
}

hipError_t launch_exchange_probe(unsigned long long* flags, int G, int block, long long steps, long long wait_ticks,
                                 unsigned* err, hipStream_t s) {
  if (G < 1 || G > kPersistMaxBlock || block < 64 || block > kPersistMaxBlock || block % 64) return hipErrorInvalidValue;
  if (G <= 256)
    hipLaunchKernelGGL(k_exchange_probe<4>, dim3(G), dim3(block), 0, s, flags, G, steps, wait_ticks, err);
  else
    hipLaunchKernelGGL(k_exchange_probe<8>, dim3(G), dim3(block), 0, s, flags, G, steps, wait_ticks, err);
  return hipGetLastError();
}

// Packed rows: row i's synapses reordered by target workgroup, the workgroups
// in XCD order, as (delay * B + local target) * 8 << 32 | weight (the byte
// offset into the LDS window from the spike's slot; in the row's order inside
// a sub-row); off[i][q] = first entry of the workgroup at place q,
// off[i][G] = the row's length.  One workgroup per row: a histogram over the
// target workgroups, its two prefix sums (target order and XCD order), then
// every entry to its place.
constexpr int kPackBlock = 256;
__global__ __launch_bounds__(kPackBlock) void k_pack_rows(const int64_t* row_ptr, const int32_t* tgt, const int32_t* wq,
                                                          const uint8_t* dly, int G, int B, unsigned* off,
                                                          unsigned long long* pk) {
  __shared__ int s_cnt[kPersistMaxBlock];     // entries per workgroup, then its shift: place in the packed row - place in the row
  __shared__ int s_wave[2][kPackBlock / 64];
  const long long i = blockIdx.x;
  const long long b = row_ptr[i];
  const int len = (int)(row_ptr[i + 1] - b);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int k = tid; k < G; k += kPackBlock) s_cnt[k] = 0;
  __syncthreads();
  for (int k = tid; k < len; k += kPackBlock) atomicAdd(&s_cnt[tgt[b + k] / B], 1);
  __syncthreads();
  // thread t takes workgroups 2t, 2t+1 in target order, and places 2t, 2t+1 in XCD order
  auto wg_at = [&](int q) {                    // workgroup at place q
    int x = 0, c = (G + kXcds - 1) / kXcds;
    while (q >= c) { q -= c; ++x; c = (G - x + kXcds - 1) / kXcds; }
    return q * kXcds + x;
  };
  int tc[2], qc[2], qg[2];
  for (int u = 0; u < 2; ++u) {
    const int k = 2 * tid + u;
    tc[u] = (k < G) ? s_cnt[k] : 0;
    qg[u] = (k < G) ? wg_at(k) : 0;
    qc[u] = (k < G) ? s_cnt[qg[u]] : 0;
  }
  const int ti = wave_incl(tc[0] + tc[1]), qi = wave_incl(qc[0] + qc[1]);
  if (lane == 63) { s_wave[0][wave] = ti; s_wave[1][wave] = qi; }
  __syncthreads();
  int t0 = ti - tc[0] - tc[1], q0 = qi - qc[0] - qc[1];
  for (int w = 0; w < wave; ++w) { t0 += s_wave[0][w]; q0 += s_wave[1][w]; }
  // every thread has read its counts: the array now takes -(first entry in the row)
  for (int u = 0; u < 2; ++u) {
    const int k = 2 * tid + u;
    if (k < G) s_cnt[k] = -(t0 + (u ? tc[0] : 0));
  }
  __syncthreads();
  for (int u = 0; u < 2; ++u) {
    const int k = 2 * tid + u;
    if (k < G) {
      const int at = q0 + (u ? qc[0] : 0);
      off[(size_t)i * (G + 1) + k] = (unsigned)at;
      s_cnt[qg[u]] += at;                      // one thread per workgroup
    }
  }
  if (tid == 0) off[(size_t)i * (G + 1) + G] = (unsigned)len;
  __syncthreads();
  for (int k = tid; k < len; k += kPackBlock) {
    const int t = tgt[b + k], g = t / B;
    pk[b + k + s_cnt[g]] = (unsigned long long)(8u * ((unsigned)dly[b + k] * (unsigned)B + (unsigned)(t - g * B))) << 32 |
                           (unsigned)wq[b + k];
  }
}

size_t persist_lds_bytes(int B, int DL) {
  const int BW = (B + 31) / 32;
  return (size_t)DL * B * 8 + (size_t)128 * BW * 4 + (size_t)kQueue * 4 + (size_t)(kPersistThreads / 64) * kUnits * 16;
}

// The instances of k_persist (recording, timing, poll width); shapes are
// checked against all of them.
const void* const kPersistFns[8] = {
    (const void*)k_persist<false, false, 4>, (const void*)k_persist<true, false, 4>,
    (const void*)k_persist<false, true, 4>,  (const void*)k_persist<true, true, 4>,
    (const void*)k_persist<false, false, 8>, (const void*)k_persist<true, false, 8>,
    (const void*)k_persist<false, true, 8>,  (const void*)k_persist<true, true, 8>};

hipError_t persist_static_lds(size_t* bytes) {
  *bytes = 0;
  for (const void* f : kPersistFns) {
    hipFuncAttributes attr;
    const hipError_t e = hipFuncGetAttributes(&attr, f);
    if (e != hipSuccess) return e;
    *bytes = std::max<size_t>(*bytes, attr.sharedSizeBytes);
  }
  return hipSuccess;
}

hipError_t persist_occupancy(int block, size_t lds, int* blocks_per_cu) {
  *blocks_per_cu = 1 << 30;
  for (const void* f : kPersistFns) {
    int occ = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, f, block, lds);
    if (e != hipSuccess) return e;
    *blocks_per_cu = std::min(*blocks_per_cu, occ);
  }
  return hipSuccess;
}

template <bool kRec, bool kTime>
static void launch_persist_as(const DevNet& p, const PersistArgs& a, int steps, int block, size_t lds, hipStream_t s) {
  auto* const kf = (a.G <= 256) ? k_persist<kRec, kTime, 4> : k_persist<kRec, kTime, 8>;
  hipLaunchKernelGGL(kf, dim3(a.G), dim3(block), lds, s, p, a, steps);
}

hipError_t launch_persist(const DevNet& p, const PersistArgs& a, int steps, int block, hipStream_t s) {
  const size_t lds = persist_lds_bytes(a.B, a.DL);
  const bool rec = p.xrec != nullptr || p.ck_y != nullptr, tim = a.phase != nullptr;
  if (rec && tim) launch_persist_as<true, true>(p, a, steps, block, lds, s);
  else if (rec) launch_persist_as<true, false>(p, a, steps, block, lds, s);
  else if (tim) launch_persist_as<false, true>(p, a, steps, block, lds, s);
  else launch_persist_as<false, false>(p, a, steps, block, lds, s);
  return hipGetLastError();
}

hipError_t launch_pack_rows(const int64_t* row_ptr, const int32_t* tgt, const int32_t* wq, const uint8_t* dly,
                            long long n_pad, int G, int B, unsigned* off, unsigned long long* pk, hipStream_t s) {
  if (G < 1 || G > kPersistMaxBlock || 2 * kPackBlock < G) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pack_rows, dim3((unsigned)n_pad), dim3(kPackBlock), 0, s, row_ptr, tgt, wq, dly, G, B, off, pk);
  return hipGetLastError();
}

hipError_t persist_set_lds_limit(size_t lds) {
  for (const void* f : kPersistFns) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mc
