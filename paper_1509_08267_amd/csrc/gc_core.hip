// gc_core.hip -- the last rounds of a colouring, or all rounds of a small graph,
// in one launch.
//
// Once at most kCoreMax vertices are uncoloured, a round's work is tiny and its
// cost is the launches and the dependent loads of each pass (20 to 60 us per
// round on a power-law graph, for some two hundred rounds).  Only the edges
// among those vertices still matter, and they fit the LDS of a few compute
// units: the core vertices are numbered 0 .. N-1 in id order, workgroup g
// takes vertices 64 g .. 64 g + 63 and keeps for each of them
//   - its row of the N x N adjacency bit matrix,
//   - the 512-bit mask of the colours final on a neighbour,
// built once from the CSR rows.  A round is then
//   1. each uncoloured vertex's least free colour; the workgroup publishes its
//      64 tentative colours, and reads everybody's;
//   2. per tentative colour of its own vertices, the bit set of the vertices
//      that carry it; a vertex loses when its row meets its colour's set below
//      itself; the workgroup publishes its winners, and reads everybody's;
//   3. each winner's colour into the masks of its own vertices (a column of
//      the matrix, by symmetry a bit of each row).
// The two exchanges are the round's only communication.  Every published word
// carries its round, so that a reader polls the data itself and no separate
// barrier is needed; a workgroup publishes a word again only after everybody
// has published the other kind in between, hence has read the earlier one, so
// one buffer of each suffices.  The words are relaxed agent-scope atomics.
//
// Every workgroup waits for all the others, so all of them have to be resident
// together: at most 64 workgroups of about 80 KB, two to a compute unit, so that
// eight such launches fit 256 compute units, more than the four kernels a process
// runs at once on its hardware queues.  Several processes may have more, or other
// kernels may keep the rest of a launch from starting for long: every wait is
// bounded (abort flag), and the vertices of a pass that gave up are coloured by the
// finishing kernel (color_alone).
//
// Bound by the two exchanges, about 2 us each. Measured, whole calls: R-MAT of
// scale 22 (the last 202 of 315 rounds) 20.7 -> 15.9 ms, 8,000 vertices and 4 M
// edges (the last 100 of 175) 3.83 -> 2.74 ms, 3,000 vertices and 300,000 edges
// (all 52) 2.16 -> 0.40 ms.
//
// Colours from 512 on have no mask bit: the pass then gives up (core_fail) and
// the caller colours the graph without it.  It looks only at calls that search
// for the round count; with that known, so are the colours, and the pass is not
// taken where they are too many.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>

#include "gc_device.h"
#include "gc_internal.h"

namespace gc {

namespace {

constexpr int kCoreBlock = 1024;
constexpr int kCoreWaves = kCoreBlock / kWave;
constexpr int kCoreWords = kCoreMax / kWave;  // 64-bit words of a matrix row at most
constexpr int kCorePitch = kCoreWords + 1;    // (padded: equal words of 64 rows on all banks)
constexpr int kMaskPitch = kCoreColors / 32 + 1;
constexpr int kNoTent = 0x3ff;   // published by a final vertex (or past the last one)
constexpr int kGaveUp = 0x3fe;   // published by a vertex with all 512 colours taken
constexpr int kLongRow = 8192;   // rows above this are built by the whole workgroup

struct CoreSmem {
  uint64_t rows[kWave][kCorePitch];
  uint64_t cls[kWave][kCorePitch];
  uint32_t mask[kWave][kMaskPitch];
  uint16_t tent[kCoreMax];
  int8_t slot[kCoreColors];  // representative lane of a tentative colour, -1 for none
  uint32_t win[2 * kCoreWords];
  uint64_t alive, lose;
  int id[kWave];
  int count, stop;
};

// Polls p until its high half carries `tag`; false when the wait was given up.
__device__ __forceinline__ bool poll(const uint64_t* p, uint32_t tag, Ctrl* c, int polls,
                                     uint64_t* out) {
  long spins = 0;
  for (;;) {
    const uint64_t x = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uint32_t)(x >> 32) == tag) {
      *out = x;
      return true;
    }
    if (++spins >= polls)
      __hip_atomic_store(&c->abort.v, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((spins & 1023) == 0 &&
        __hip_atomic_load(&c->abort.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return false;
  }
}

// One row entry of own vertex i: a final neighbour's colour into its mask, an
// uncoloured one (a core vertex) into its matrix row.
template <typename S>
__device__ __forceinline__ void build_entry(const KArgs& a, CoreSmem& sm, int i, int u) {
  const int s = ((const S*)a.st)[u];
  if (s < 0) {
    const int x = a.skip[u];
    atomicOr((uint32_t*)&sm.rows[i][x >> 6] + ((x >> 5) & 1), 1u << (x & 31));
  } else if (s < kCoreColors) {
    atomicOr(&sm.mask[i][s >> 5], 1u << (s & 31));
  }
}

template <typename S, typename RP>
__device__ __forceinline__ void build_row(const KArgs& a, CoreSmem& sm, int i, RP b, RP e, int tid,
                                          int step) {
  for (RP k = b + tid; k < e; k += 4 * (RP)step) {
    int u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) u[j] = k + j * step < e ? a.colidx[k + j * step] : -1;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (u[j] >= 0) build_entry<S>(a, sm, i, u[j]);
  }
}

// Rounds round0 + 1, ... until no core vertex is uncoloured, or (last > 0)
// round `last` has run.
template <typename RP, typename S>
__global__ __launch_bounds__(kCoreBlock) void k_core(KArgs a, CoreArgs c, int round0,
                                                     int last) {
  extern __shared__ __align__(16) char smem_raw[];
  CoreSmem& sm = *(CoreSmem*)smem_raw;
  const RP* __restrict__ rp = (const RP*)a.rowptr;
  S* __restrict__ st = (S*)a.st;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int g = blockIdx.x;
  const int N = a.ctrl->core_n.v;
  // more core vertices than the launch was sized for (the graph changed): none
  // of the workgroups starts
  if (N > (int)gridDim.x * kWave) {
    if (tid == 0) a.ctrl->core_fail.v = 1;
    return;
  }
  const int nw = gridDim.x;  // 64-bit words of a row
  const int own = min(kWave, max(0, N - g * kWave));
  for (int i = tid; i < kWave * kCorePitch; i += kCoreBlock) (&sm.rows[0][0])[i] = 0;
  for (int i = tid; i < kWave * kMaskPitch; i += kCoreBlock) (&sm.mask[0][0])[i] = 0;
  if (tid < kWave) sm.id[tid] = tid < own ? c.ids[g * kWave + tid] : -1;
  if (tid == 0) {
    sm.alive = own == kWave ? ~0ull : (1ull << own) - 1;
    sm.stop = 0;
  }
  __syncthreads();
  for (int i = wave; i < own; i += kCoreWaves) {
    const int v = sm.id[i];
    const RP b = rp[v], e = rp[v + 1];
    if (e - b <= (RP)kLongRow) build_row<S, RP>(a, sm, i, b, e, lane, kWave);
  }
  for (int i = 0; i < own; ++i) {
    const int v = sm.id[i];
    const RP b = rp[v], e = rp[v + 1];
    if (e - b > (RP)kLongRow) build_row<S, RP>(a, sm, i, b, e, tid, kCoreBlock);
  }
  __syncthreads();
  int t = 0;  // wave 0: this lane's tentative colour
  int rounds = 0;
  for (uint32_t q = 1;; ++q) {  // q: the round's tag
    // 1. tentative colours
    if (wave == 0) {
      const bool mine = (sm.alive >> lane) & 1;
      if (mine) {
        uint32_t free = 0;
        int w = t >> 5;
        for (; w < kCoreColors / 32; ++w) {
          free = ~sm.mask[lane][w] & (w == t >> 5 ? ~0u << (t & 31) : ~0u);
          if (free) break;
        }
        t = free ? 32 * w + __builtin_ctz(free) : kGaveUp;
      }
      // two vertices of one word: the even lane publishes both
      const int x = mine ? t : kNoTent;
      const int y = __shfl_xor(x, 1);
      if ((lane & 1) == 0)
        __hip_atomic_store(&c.tents[(g * kWave + lane) >> 1],
                           ((uint64_t)q << 32) | (uint32_t)(x | (y << 16)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int i = tid; i < kWave * kCorePitch; i += kCoreBlock) (&sm.cls[0][0])[i] = 0;
    for (int i = tid; i < kCoreColors; i += kCoreBlock) sm.slot[i] = -1;
    if (tid == 0) {
      sm.lose = 0;
      sm.count = 0;
    }
    int left = 0, bad = 0;
    for (int i = tid; i < nw * (kWave / 2); i += kCoreBlock) {
      uint64_t x = 0;
      if (!poll(&c.tents[i], q, a.ctrl, c.polls, &x)) bad = 1;
      const int x0 = (int)(x & 0xffff), x1 = (int)((x >> 16) & 0xffff);
      sm.tent[2 * i] = (uint16_t)x0;
      sm.tent[2 * i + 1] = (uint16_t)x1;
      left += (x0 != kNoTent) + (x1 != kNoTent);
      if (x0 == kGaveUp || x1 == kGaveUp) {  // (every workgroup reads the same words)
        a.ctrl->core_fail.v = 1;
        bad = 1;
      }
    }
    if (__syncthreads_or(bad)) return;
    if (!__syncthreads_or(left) || (last > 0 && round0 + rounds >= last)) break;
    ++rounds;
    if (g == 0) {  // |U_r|, by workgroup 0
#pragma unroll
      for (int off = kWave / 2; off > 0; off >>= 1) left += __shfl_xor(left, off);
      if (lane == 0 && left) atomicAdd(&sm.count, left);
    }
    // 2. the sets of the own vertices' colours, and the conflicts
    const int mt = sm.tent[g * kWave + lane];  // (of the lane's vertex, in every wavefront)
    const bool mine = mt < kCoreColors;
    if (wave == 0 && mine) sm.slot[mt] = (int8_t)lane;
    __syncthreads();
    if (g == 0 && tid == 0) {
      const int r = round0 + rounds;
      if (r <= kTraceRounds) a.ctrl->trace[r - 1] = sm.count;
    }
    for (int v = tid; v < (g + 1) * kWave; v += kCoreBlock) {
      const int tv = sm.tent[v];
      if (tv < kCoreColors) {
        const int s = sm.slot[tv];
        if (s >= 0) atomicOr((uint32_t*)&sm.cls[s][v >> 6] + ((v >> 5) & 1), 1u << (v & 31));
      }
    }
    __syncthreads();
    bool lose = false;
    if (mine) {
      const int s = sm.slot[mt];
      for (int w = wave; w <= g; w += kCoreWaves) {
        const uint64_t below = w < g ? ~0ull : (1ull << lane) - 1;
        lose |= (sm.cls[s][w] & sm.rows[lane][w] & below) != 0;
      }
    }
    const uint64_t lm = __ballot(lose);
    if (lane == 0 && lm) atomicOr((unsigned long long*)&sm.lose, (unsigned long long)lm);
    __syncthreads();
    const uint64_t won = sm.alive & ~sm.lose;
    if (wave == 0) {
      if (lane < 2)
        __hip_atomic_store(&c.wins[2 * g + lane],
                           ((uint64_t)q << 32) | (uint32_t)(won >> (32 * lane)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      if ((won >> lane) & 1) st[sm.id[lane]] = (S)t;
    }
    bad = 0;
    if (tid < 2 * nw) {
      uint64_t x = 0;
      if (!poll(&c.wins[tid], q, a.ctrl, c.polls, &x)) bad = 1;
      sm.win[tid] = (uint32_t)x;
    }
    if (__syncthreads_or(bad)) return;
    // 3. the winners' colours
    if (tid == 0) sm.alive &= ~won;
    for (int j = wave; j < 2 * nw; j += kCoreWaves) {
      uint32_t m = sm.win[j];
      while (m) {  // wave-uniform
        const int v = 32 * j + __builtin_ctz(m);
        m &= m - 1;
        const int col = sm.tent[v];
        if ((sm.rows[lane][v >> 6] >> (v & 63)) & 1)
          atomicOr(&sm.mask[lane][col >> 5], 1u << (col & 31));
      }
    }
    __syncthreads();
  }
  if (g == 0 && tid == 0 && rounds > 0) a.ctrl->last_round.v = round0 + rounds;
}

// The uncoloured vertices in id order.  Workgroup b of kCoreGrid takes a
// contiguous range of vertices; phase 0 counts into part[b], phase 1 writes
// the ids behind those of the workgroups before it (none if there are more
// than kCoreMax), each vertex's number into skip, and clears the exchange words.
template <typename S>
__global__ __launch_bounds__(kBlock) void k_core_collect(KArgs a, CoreArgs c, int phase) {
  __shared__ int cnt[kWavesPerBlock];
  const S* __restrict__ st = (const S*)a.st;
  const long nchunks = ((long)a.n + kWave - 1) / kWave;
  const long per = (nchunks + gridDim.x - 1) / gridDim.x;
  const long c0 = min(nchunks, (long)blockIdx.x * per), c1 = min(nchunks, c0 + per);
  const int wave = threadIdx.x / kWave, lane = lane_id();
  auto open = [&](long ch) {
    const long v = ch * kWave + lane;
    return __ballot(ch < c1 && v < a.n && st[v < a.n ? v : 0] < 0);
  };
  if (phase == 0) {
    if (blockIdx.x == 0) fold_trace(a.ctrl, a.part);  // the last detect pass's round size
    int mine = 0;
    for (long ch = c0 + wave; ch < c1; ch += kWavesPerBlock) mine += __popcll(open(ch));
    if (lane == 0) cnt[wave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < kWavesPerBlock; ++w) mine += cnt[w];
      c.part[blockIdx.x] = mine;
    }
    return;
  }
  int at = 0, all = 0;
  for (int b = 0; b < (int)gridDim.x; ++b) {
    at += b < (int)blockIdx.x ? c.part[b] : 0;
    all += c.part[b];
  }
  const long tid = blockIdx.x * (long)blockDim.x + threadIdx.x;
  const long nth = (long)gridDim.x * blockDim.x;
  for (long i = tid; i < kCoreMax / 2; i += nth) c.tents[i] = 0;
  for (long i = tid; i < 2 * kCoreWords; i += nth) c.wins[i] = 0;
  if (tid == 0) a.ctrl->core_n.v = all;
  if (all > kCoreMax) return;
  for (long cb = c0; cb < c1; cb += kWavesPerBlock) {  // workgroup-uniform
    const uint64_t m = open(cb + wave);
    if (lane == 0) cnt[wave] = __popcll(m);
    __syncthreads();
    int before = 0, sum = 0;
    for (int w = 0; w < kWavesPerBlock; ++w) {
      before += w < wave ? cnt[w] : 0;
      sum += cnt[w];
    }
    if ((m >> lane) & 1) {
      const int i = at + before + __popcll(m & ((1ull << lane) - 1));
      const int v = (int)((cb + wave) * kWave) + lane;
      c.ids[i] = v;
      a.skip[v] = i;
    }
    at += sum;
    __syncthreads();
  }
}

template <typename RP, typename S>
int launch_core_t(const KArgs& a, const CoreArgs& c, int round0, int last, int workgroups,
                  hipStream_t s) {
  static_assert(sizeof(CoreSmem) <= 80 * 1024, "two workgroups per compute unit");
  const int rc = allow_lds((const void*)&k_core<RP, S>, (int)sizeof(CoreSmem));
  if (rc) return rc;
  hipLaunchKernelGGL((k_core<RP, S>), dim3(workgroups), dim3(kCoreBlock), sizeof(CoreSmem), s, a, c,
                     round0, last);
  return (int)hipGetLastError();
}

}  // namespace

int launch_core_collect(const KArgs& a, int sbytes, const CoreArgs& c, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const long chunks = ((long)a.n + kWave - 1) / kWave;
  const int grid = (int)std::max<long>(
      1, std::min<long>(kCoreGrid, (chunks + kWavesPerBlock - 1) / kWavesPerBlock));
  for (int phase = 0; phase < 2; ++phase) {
    if (sbytes == 1)
      hipLaunchKernelGGL((k_core_collect<int8_t>), dim3(grid), dim3(kBlock), 0, s, a, c, phase);
    else if (sbytes == 2)
      hipLaunchKernelGGL((k_core_collect<int16_t>), dim3(grid), dim3(kBlock), 0, s, a, c, phase);
    else
      hipLaunchKernelGGL((k_core_collect<int32_t>), dim3(grid), dim3(kBlock), 0, s, a, c, phase);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
  }
  return 0;
}

int launch_core(const KArgs& a, bool rp64, int sbytes, const CoreArgs& c, int round0, int last,
                int workgroups, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  if (workgroups < 1 || workgroups > kCoreWords) return (int)hipErrorInvalidValue;
#define GC_CORE(S_)                                                                 \
  return rp64 ? launch_core_t<int64_t, S_>(a, c, round0, last, workgroups, s)             \
              : launch_core_t<int32_t, S_>(a, c, round0, last, workgroups, s)
  if (sbytes == 1) GC_CORE(int8_t);
  if (sbytes == 2) GC_CORE(int16_t);
  GC_CORE(int32_t);
#undef GC_CORE
}

}  // namespace gc
