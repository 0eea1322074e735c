// gc_seq.hip -- sequential First Fit (GC_ALGO_SEQ) in one launch, by data flow.
//
// The id-priority schedule colours a vertex in the first round in which all
// its lower-id neighbours are coloured.  Its colour (the least one absent
// from the lower neighbours) and its round (one more than the largest of
// theirs) depend on those neighbours alone, so no barrier is needed between
// the rounds: a vertex is coloured as soon as its lower neighbours are, and
// the round is carried along with the colour in one word per vertex,
//   0                          not coloured yet
//   (round << cbits) | colour  final.
// A launch per round visits every waiting vertex every round (the longest
// id-increasing path sets their number: 94 rounds on a uniform random graph of
// 2^20 vertices and 2^24 edges, over a thousand on a power-law one); here each
// row's lower prefix is read once, and a vertex waits only for what it needs.
// Measured, whole call: uniform random graph of 2^20 vertices and 2^24 edges
// 3.44 -> 0.32 ms, R-MAT of scale 20 and edge factor 16 71.6 -> 2.2 ms.  What
// is left is the chain itself, about 1.8 us per round: a store, the polling
// load that sees it, the pick.
//
// Mapping: units of consecutive ids (at most 64 vertices of small degree, or
// one vertex of degree above light_max) are handed to wavefronts in id order
// by a ticket.  A light unit's vertices take a lane each, a larger vertex the
// whole wavefront; kFlow entries per lane are polled at a time.  Every
// dependency of a unit lies in the unit itself or in one with a smaller
// ticket, and a wavefront never blocks inside a unit (its lanes advance
// independently in one polling loop), so the lowest vertex not yet coloured is
// always held by a running wavefront: the kernel drains whatever the number of
// resident wavefronts.  A group of L lanes per light vertex was slower the
// wider it was (the 2^24-edge graph: L = 1 331 us, 2 599, 4 1,121, 8 2,440): a
// group works on its vertices in turn, and a waiting one holds up the rest.
// Four entries per lane in flight: 331 us, two 373, eight 331, sixteen 352.
//
// Visibility: a word is one naturally atomic store and says everything a
// reader needs, so relaxed agent-scope stores and loads suffice.  The first
// look at a neighbour is an ordinary cached load (a final word never
// changes, and a stale one only reads "not yet"); repeated looks are
// agent-scope loads.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>

#include "gc_device.h"
#include "gc_internal.h"

namespace gc {

namespace {

constexpr int kFlow = 4;               // row entries per lane polled together
constexpr int kFlowBits = 1024;        // colour window of a wavefront-wide vertex (LDS bits)
constexpr int kFlowBins = 2048;        // rounds counted in LDS by the finishing pass
constexpr long kFlowSpinLimit = 1l << 25;

template <typename W>
__device__ __forceinline__ W look(const W* p, bool first) {
  return first ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)
               : __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Idle polling: after a pass over a wavefront's entries that changed nothing,
// pause; give up (setting the abort flag) only far beyond any wait of a
// graph that fits a GPU.  Returns whether to stop.
__device__ __forceinline__ bool idle(Ctrl* c, long& spins) {
  __builtin_amdgcn_s_sleep(1);
  if (++spins > kFlowSpinLimit) {
    __hip_atomic_store(&c->abort.v, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
  }
  return (spins & 1023) == 0 &&
         __hip_atomic_load(&c->abort.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// The largest x of the wavefront, in every lane (x >= 0).  Row shifts and row
// broadcasts: a chain of register moves, where a shuffle would add an LDS
// access per step to every link of the dependency chain.
__device__ __forceinline__ int wave_max(int x) {
#define GC_MAX_STEP(ctrl, rows)                                                  \
  {                                                                              \
    const int y = __builtin_amdgcn_update_dpp(0, x, ctrl, rows, 0xf, false);     \
    x = y > x ? y : x;                                                           \
  }
  GC_MAX_STEP(0x111, 0xf);  // row_shr:1, :2, :4, :8
  GC_MAX_STEP(0x112, 0xf);
  GC_MAX_STEP(0x114, 0xf);
  GC_MAX_STEP(0x118, 0xf);
  GC_MAX_STEP(0x142, 0xa);  // row_bcast:15 into rows 1 and 3
  GC_MAX_STEP(0x143, 0xc);  // row_bcast:31 into rows 2 and 3
#undef GC_MAX_STEP
  return __builtin_amdgcn_readlane(x, kWave - 1);
}

constexpr int kDeepWords = 8;
constexpr int kDeepBits = 32 * kDeepWords;
constexpr int kDeepPitch = kDeepWords + 1;

// First clear bit of a lane's LDS words, -1 for none.
__device__ __forceinline__ int deep_free(const uint32_t* more) {
  int c = -1;
#pragma unroll
  for (int q = kDeepWords - 1; q >= 0; --q) {
    const uint32_t x = more[q];
    if (x != ~0u) c = 32 * q + __builtin_ctz(~x);
  }
  return c;
}

// The vertices s0 .. s0 + cnt - 1 (cnt <= 64), one per lane.  The loop is
// wave-uniform and every lane keeps its own place in its own row, so no lane
// waits inside it.  Returns whether to stop (abort).  A lane holds the taken
// colours of a window of 64 and walks its row again for the next one.  Where a lane
// walks rows of more than 64 entries (DEEP) the window goes on for kDeepBits colours
// in LDS (deep, this wavefront's own): a second walk took ten times as long as a
// link of the chain (200 cliques of 200 vertices 7.5 ms, now 0.28; four words in
// registers cost uniform random graphs of such degrees 10 to 20%).
template <typename RP, typename W, bool DEEP>
__device__ bool flow_light(const FlowArgs& a, int s0, int cnt, uint32_t* deep) {
  const RP* __restrict__ rp = (const RP*)a.rowptr;
  W* const word = (W*)a.word;
  const W cmask = ((W)1 << a.cbits) - 1;
  const int v = s0 + lane_id();
  bool alive = lane_id() < cnt;
  const RP b = alive ? rp[v] : 0, e = alive ? rp[v + 1] : 0;
  RP k = b;
  int base = 0;
  bool fetch = true, first = false, past = false;
  int pend = 0;  // bit j: entry u[j] is not yet final
  int u[kFlow] = {};
  uint64_t m = 0;
  uint32_t* const more = deep + lane_id() * kDeepPitch;
  if (DEEP)
    for (int q = 0; q < kDeepWords; ++q) more[q] = 0;
  int top = 0;  // largest round among the lower neighbours
  long spins = 0;
  while (__ballot(alive)) {
    bool moved = false;
    if (alive && fetch) {
#pragma unroll
      for (int j = 0; j < kFlow; ++j) u[j] = k + j < e ? a.colidx[k + j] : INT32_MAX;
      past = k + kFlow >= e;
#pragma unroll
      for (int j = 0; j < kFlow; ++j) {
        pend |= (u[j] < v) << j;
        past |= a.sorted && u[j] >= v;
      }
      k += kFlow;
      fetch = false;
      first = true;
      moved = true;
    }
    if (pend) {
      W w[kFlow];
#pragma unroll
      for (int j = 0; j < kFlow; ++j) w[j] = (pend >> j) & 1 ? look(&word[u[j]], first) : (W)0;
#pragma unroll
      for (int j = 0; j < kFlow; ++j)
        if (w[j]) {
          pend &= ~(1 << j);
          const unsigned rel = (unsigned)(w[j] & cmask) - (unsigned)base;
          if (rel < 64u) m |= 1ull << rel;
          else if (DEEP && rel < 64u + kDeepBits) more[(rel - 64u) >> 5] |= 1u << (rel & 31);
          top = max(top, (int)(w[j] >> a.cbits));
          moved = true;
        }
      first = false;
    }
    if (alive && !pend) {
      // (the first window at once: this is the chain's own link)
      if (!past) {
        fetch = true;
      } else if (m != ~0ull) {
        const W x = ((W)(top + 1) << a.cbits) | (W)(base + __builtin_ctzll(~m));
        __hip_atomic_store(&word[v], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        alive = false;
      } else if (const int c = DEEP ? deep_free(more) : -1; c >= 0) {
        const W x = ((W)(top + 1) << a.cbits) | (W)(base + 64 + c);
        __hip_atomic_store(&word[v], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        alive = false;
      } else {  // the whole window is taken: slide it
        base += 64 + (DEEP ? kDeepBits : 0);
        m = 0;
        if (DEEP)
          for (int q = 0; q < kDeepWords; ++q) more[q] = 0;
        k = b;
        fetch = true;
      }
      moved = true;
    }
    if (__ballot(moved)) spins = 0;
    else if (idle(a.ctrl, spins)) return true;
  }
  return false;
}

// One vertex by the whole wavefront; its forbidden colours meet in an LDS
// bitmap of kFlowBits (bm, this wavefront's own).
template <typename RP, typename W>
__device__ bool flow_wave(const FlowArgs& a, int v, RP b, RP e, uint32_t* bm) {
  const int lane = lane_id();
  W* const word = (W*)a.word;
  const W cmask = ((W)1 << a.cbits) - 1;
  long spins = 0;
  for (int base = 0;; base += kFlowBits) {
    if (lane < kFlowBits / 32) bm[lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    int top = 0;
    bool past = false;
    for (RP kb = b; kb < e && !past; kb += kFlow * kWave) {  // wave-uniform
      int u[kFlow], pend = 0;
      bool mine = false;
#pragma unroll
      for (int j = 0; j < kFlow; ++j) {
        const RP p = kb + j * kWave + lane;
        u[j] = p < e ? a.colidx[p] : INT32_MAX;
      }
#pragma unroll
      for (int j = 0; j < kFlow; ++j) {
        pend |= (u[j] < v) << j;
        mine |= a.sorted && u[j] >= v;
      }
      past = __ballot(mine) != 0;
      bool first = true;
      while (__ballot(pend != 0)) {
        bool moved = first;
        W w[kFlow];
#pragma unroll
        for (int j = 0; j < kFlow; ++j) w[j] = (pend >> j) & 1 ? look(&word[u[j]], first) : (W)0;
#pragma unroll
        for (int j = 0; j < kFlow; ++j)
          if (w[j]) {
            pend &= ~(1 << j);
            const unsigned rel = (unsigned)(w[j] & cmask) - (unsigned)base;
            if (rel < (unsigned)kFlowBits) atomicOr(&bm[rel >> 5], 1u << (rel & 31));
            top = max(top, (int)(w[j] >> a.cbits));
            moved = true;
          }
        first = false;
        if (__ballot(moved)) spins = 0;
        else if (idle(a.ctrl, spins)) return true;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    const uint32_t x = lane < kFlowBits / 32 ? bm[lane] : ~0u;
    const uint64_t open = __ballot(x != ~0u);
    top = wave_max(top);
    if (!open) continue;  // the whole window is taken: slide it
    const int q = __builtin_ctzll(open);
    const uint32_t y = (uint32_t)__builtin_amdgcn_readlane((int)x, q);
    const W c = (W)(base + 32 * q + __builtin_ctz(~y));
    if (lane == 0)
      __hip_atomic_store(&word[v], ((W)(top + 1) << a.cbits) | c, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    return false;
  }
}

template <typename RP, typename W, bool DEEP>
__global__ __launch_bounds__(kBlock) void k_seq_flow(FlowArgs a) {
  __shared__ uint32_t deep[kWavesPerBlock][DEEP ? kWave * kDeepPitch : 1];
  __shared__ uint32_t bitmap[kWavesPerBlock][kFlowBits / 32];
  const RP* __restrict__ rp = (const RP*)a.rowptr;
  const int units = *a.units;
  for (;;) {
    int t = 0;
    if (lane_id() == 0) t = atomicAdd(&a.ctrl->ticket.v, 1);
    t = __shfl(t, 0);
    if (t >= units) break;  // wave-uniform
    const int s0 = a.starts[t], s1 = a.starts[t + 1];
    bool stop;
    if (s1 - s0 == 1 && rp[s0 + 1] - rp[s0] > (RP)a.light_max)
      stop = flow_wave<RP, W>(a, s0, rp[s0], rp[s0 + 1], bitmap[threadIdx.x / kWave]);
    else
      stop = flow_light<RP, W, DEEP>(a, s0, s1 - s0, deep[threadIdx.x / kWave]);
    if (stop) break;
  }
}

template <typename W>
__global__ __launch_bounds__(kBlock) void k_flow_clear(FlowArgs a) {
  W* const word = (W*)a.word;
  const long tid = blockIdx.x * (long)blockDim.x + threadIdx.x;
  const long nth = (long)gridDim.x * blockDim.x;
  for (long v = tid; v < a.n; v += nth) word[v] = 0;
}

// The words become the caller's colours, and the call's statistics: per
// workgroup the largest colour and the uncoloured count (as the finishing
// pass of the rounds), the largest round, and |U_r| = the vertices of round
// r or later.  The rounds are counted per workgroup in LDS (the first
// kFlowBins of them) and added into the trace; the workgroup that finishes
// last turns the counts into suffix sums.
template <typename W>
__global__ __launch_bounds__(kBlock) void k_flow_finish(FlowArgs a, int32_t* out) {
  __shared__ int bins[kFlowBins];
  __shared__ int part[kBlock];
  __shared__ int sh_max[kWavesPerBlock], sh_left[kWavesPerBlock], sh_round[kWavesPerBlock];
  __shared__ int last;
  const W* __restrict__ word = (const W*)a.word;
  const W cmask = ((W)1 << a.cbits) - 1;
  for (int i = threadIdx.x; i < kFlowBins; i += kBlock) bins[i] = 0;
  __syncthreads();
  int mx = -1, left = 0, round = 0, over = 0;
  const long tid = blockIdx.x * (long)blockDim.x + threadIdx.x;
  const long nth = (long)gridDim.x * blockDim.x;
  for (long v = tid; v < a.n; v += nth) {
    W w = word[v];
    if (a.last > 0 && (w >> a.cbits) > (W)a.last) w = 0;
    const int c = w ? (int)(w & cmask) : -1;
    const int r = (int)(w >> a.cbits);
    a.colors[v] = c;
    mx = max(mx, c);
    left += w == 0;
    round = max(round, r);
    if (r > kTraceRounds) ++over;
    else if (r > kFlowBins) atomicAdd(&a.ctrl->trace[r - 1], 1);
    else if (r > 0) atomicAdd(&bins[r - 1], 1);
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    mx = max(mx, __shfl_xor(mx, off));
    round = max(round, __shfl_xor(round, off));
    left += __shfl_xor(left, off);
    over += __shfl_xor(over, off);
  }
  if (lane_id() == 0) {
    sh_max[threadIdx.x / kWave] = mx;
    sh_left[threadIdx.x / kWave] = left;
    sh_round[threadIdx.x / kWave] = round;
    if (over) atomicAdd(&a.ctrl->over.v, over);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kFlowBins; i += kBlock)
    if (bins[i]) atomicAdd(&a.ctrl->trace[i], bins[i]);
  if (threadIdx.x == 0) {
    for (int w = 1; w < kWavesPerBlock; ++w) {
      mx = max(mx, sh_max[w]);
      left += sh_left[w];
      round = max(round, sh_round[w]);
    }
    store_system(&out[kFinishHeader + 2 * blockIdx.x], mx + 1);
    store_system(&out[kFinishHeader + 1 + 2 * blockIdx.x], left);
    if (round) atomicMax(&a.ctrl->last_round.v, round);
  }
  drain_stores();  // every thread's adds
  __syncthreads();
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    last = __hip_atomic_fetch_add(&a.ctrl->bar.v, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
           (int)gridDim.x - 1;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
  if (!last) return;
  auto agent = [](const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  const int R = agent(&a.ctrl->last_round.v);
  const int T = min(R, kTraceRounds);
  const int per = (T + kBlock - 1) / kBlock;  // consecutive rounds per thread
  const int r0 = min(T, (int)threadIdx.x * per), r1 = min(T, r0 + per);
  int sum = 0;
  for (int r = r0; r < r1; ++r) sum += agent(&a.ctrl->trace[r]);
  part[threadIdx.x] = sum;
  __syncthreads();
  int after = agent(&a.ctrl->over.v);
  for (int t = threadIdx.x + 1; t < kBlock; ++t) after += part[t];
  for (int r = r1 - 1; r >= r0; --r) {
    after += agent(&a.ctrl->trace[r]);
    a.ctrl->trace[r] = after;
  }
  if (threadIdx.x == 0) {
    store_system(&out[0], R);
    store_system(&out[1], agent(&a.ctrl->abort.v));
    store_system(&out[2], 0);
    store_system(&out[3], (int32_t)gridDim.x);
    store_system(&out[4], 0);
    store_system(&out[5], -1);
    store_system(&out[6], 0);
  }
}

// ------------------------------------------------------ set-up: the units --

// First ids of the units of 64-vertex chunk ch, as a bit mask: the chunk's
// own start, every vertex of degree above light_max, and the vertex after one.
template <typename RP>
__device__ __forceinline__ uint64_t unit_starts(const RP* rp, int n, int light_max, long ch) {
  const long v = ch * kWave + lane_id();
  const bool in = v < n;
  const uint64_t big = __ballot(in && rp[v + 1] - rp[v] > (RP)light_max);
  return (1ull | big | (big << 1)) & __ballot(in);
}

// Workgroup b of kUnitGrid takes a contiguous range of chunks; phase 0 counts
// its units into part[b], phase 1 writes their first ids behind those of the
// workgroups before it.
template <typename RP>
__global__ __launch_bounds__(kBlock) void k_flow_units(FlowArgs a, int32_t* part, int32_t* starts,
                                                       int32_t* units, int phase) {
  __shared__ int cnt[kWavesPerBlock];
  const RP* rp = (const RP*)a.rowptr;
  const long nchunks = ((long)a.n + kWave - 1) / kWave;
  const long per = (nchunks + gridDim.x - 1) / gridDim.x;
  const long c0 = min(nchunks, (long)blockIdx.x * per), c1 = min(nchunks, c0 + per);
  const int wave = threadIdx.x / kWave;
  if (phase == 0) {
    int mine = 0;
    for (long c = c0 + wave; c < c1; c += kWavesPerBlock)
      mine += __popcll(unit_starts<RP>(rp, a.n, a.light_max, c));
    if (lane_id() == 0) cnt[wave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < kWavesPerBlock; ++w) mine += cnt[w];
      part[blockIdx.x] = mine;
    }
    return;
  }
  int at = 0;
  for (int b = 0; b < (int)blockIdx.x; ++b) at += part[b];
  for (long cb = c0; cb < c1; cb += kWavesPerBlock) {  // workgroup-uniform
    const long c = cb + wave;
    const uint64_t sm = c < c1 ? unit_starts<RP>(rp, a.n, a.light_max, c) : 0;
    if (lane_id() == 0) cnt[wave] = __popcll(sm);
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < kWavesPerBlock; ++w) {
      before += w < wave ? cnt[w] : 0;
      all += cnt[w];
    }
    if ((sm >> lane_id()) & 1)
      starts[at + before + __popcll(sm & ((1ull << lane_id()) - 1))] =
          (int)(c * kWave) + lane_id();
    at += all;
    __syncthreads();
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    starts[at] = a.n;
    *units = at;
  }
}

}  // namespace

int launch_flow_units(const FlowArgs& a, bool rp64, int32_t* part, int32_t* starts, int32_t* units,
                      int grid, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  for (int phase = 0; phase < 2; ++phase) {
    if (rp64)
      hipLaunchKernelGGL((k_flow_units<int64_t>), dim3(grid), dim3(kBlock), 0, s, a, part, starts,
                         units, phase);
    else
      hipLaunchKernelGGL((k_flow_units<int32_t>), dim3(grid), dim3(kBlock), 0, s, a, part, starts,
                         units, phase);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
  }
  return 0;
}

int launch_flow_clear(const FlowArgs& a, int grid, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  if (a.wide) hipLaunchKernelGGL((k_flow_clear<uint64_t>), dim3(grid), dim3(kBlock), 0, s, a);
  else hipLaunchKernelGGL((k_flow_clear<uint32_t>), dim3(grid), dim3(kBlock), 0, s, a);
  return (int)hipGetLastError();
}

int launch_flow(const FlowArgs& a, bool rp64, int grid, void* stream) {
  hipStream_t s = (hipStream_t)stream;
#define GC_FLOW(RP_, W_)                                                            \
  if (a.light_max <= 64)                                                            \
    hipLaunchKernelGGL((k_seq_flow<RP_, W_, false>), dim3(grid), dim3(kBlock), 0, s, a); \
  else                                                                              \
    hipLaunchKernelGGL((k_seq_flow<RP_, W_, true>), dim3(grid), dim3(kBlock), 0, s, a)
  if (rp64 && a.wide) {
    GC_FLOW(int64_t, uint64_t);
  } else if (rp64) {
    GC_FLOW(int64_t, uint32_t);
  } else if (a.wide) {
    GC_FLOW(int32_t, uint64_t);
  } else {
    GC_FLOW(int32_t, uint32_t);
  }
#undef GC_FLOW
  return (int)hipGetLastError();
}

int launch_flow_finish(const FlowArgs& a, int32_t* out, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const int grid =
      (int)std::max<long>(1, std::min<long>(kFinishBlocks / 2, ((long)a.n + 4 * kBlock - 1) / (4 * kBlock)));
  if (a.wide) hipLaunchKernelGGL((k_flow_finish<uint64_t>), dim3(grid), dim3(kBlock), 0, s, a, out);
  else hipLaunchKernelGGL((k_flow_finish<uint32_t>), dim3(grid), dim3(kBlock), 0, s, a, out);
  return (int)hipGetLastError();
}

}  // namespace gc
