// gc_blocks.hip -- Algorithm 1 of Section 3.1 with p blocks, read literally
// (GC_ALGO_BLOCKS).
//
// The vertices are split into p blocks of consecutive ids (block(v) =
// floor(v p / n)).  Every vertex keeps a ForbiddenColors slot per CSR entry.
// A round is
//   phase 1: each block colours its vertices still to colour, in increasing
//            id order, each with the least colour absent from its slots, and
//            writes that colour into the slot for it of every neighbour in the
//            same block;
//   phase 2: each such vertex with neighbours in other blocks copies their
//            current colours into its slots for them, and is recoloured next
//            round when one of them, in a higher-numbered block, has its
//            colour (the paper's "the vertex in the lower partition is
//            recoloured").
// Mapping: one wavefront per block in phase 1 (a block is sequential by
// definition; the wavefront searches each row for the least absent colour
// together), one wavefront per 64 consecutive vertices in phase 2, a kernel
// boundary per barrier.
//
// The slot for a neighbour in the same block always equals that
// neighbour's current colour (it is written whenever the neighbour is
// coloured, and both start at -1), so phase 1 reads the colour array for
// those entries and the slot array holds only entries whose neighbour lies
// in another block.  A colour written for a vertex is read by later vertices
// of its block in the same wavefront: a workgroup-scope fence orders the
// write before those reads.
//
// The slots themselves are not needed.  A vertex is to be recoloured in round
// r + 1 only if it was in round r, so what its slots for other blocks hold is
// always the neighbours' colours after round r's phase 1: phase 1 of the next
// round needs of them only which colours occur, and phase 2 of round r, which
// gathers those colours anyway, leaves that as a 128-bit mask per vertex (the
// k_blkm_ passes; maximum degree at most 126, so every colour has a bit).
// Phase 1 then reads no row at all: the vertices of a block without neighbours
// in their block pick in parallel, the others in turn with their block's
// colours in registers.  Larger degrees or blocks take the passes with slots.
// Bound by phase 2's colour gathers (one per entry of every vertex to
// recolour, 231 M over the 17 rounds of the uniform random graph of 2^24 edges
// with p = 16,384, in 1.1 to 1.2 ms: 200 G/s, where gathers from L2 alone reach
// 270 to 290).  That call: 4.17 ms with slots, 1.37 with masks.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "gc_device.h"
#include "gc_internal.h"

namespace gc {

// first id of block b: the least v with floor(v p / n) == b
__device__ __forceinline__ int block_start(long b, int n, long p) {
  return (int)((b * (long)n + p - 1) / p);
}

template <typename RP>
__global__ __launch_bounds__(kBlock) void k_blk_init(BArgs a) {
  const long tid = blockIdx.x * (long)blockDim.x + threadIdx.x;
  const long nth = (long)gridDim.x * blockDim.x;
  for (long v = tid; v < a.n; v += nth) {
    a.color[v] = -1;
    a.todo[v] = 1;
  }
  const long nnz = a.n > 0 ? (long)((const RP*)a.rowptr)[a.n] : 0;
  for (long k = tid; k < nnz; k += nth) a.slot[k] = -1;
}

template <typename RP>
__global__ __launch_bounds__(kBlock) void k_blk_phase1(BArgs a) {
  const RP* __restrict__ rp = (const RP*)a.rowptr;
  const int lane = lane_id();
  const long wave_gid = blockIdx.x * (long)kWavesPerBlock + threadIdx.x / kWave;
  const long nwaves = (long)gridDim.x * kWavesPerBlock;
  for (long b = wave_gid; b < a.p; b += nwaves) {
    const int v0 = block_start(b, a.n, a.p), v1 = block_start(b + 1, a.n, a.p);
    for (int v = v0; v < v1; ++v) {  // wave-uniform
      if (!a.todo[v]) continue;
      const RP rb = rp[v], re = rp[v + 1];
      int c = 0;
      for (int base = 0;; base += kWave) {  // least colour absent from the slots
        uint64_t m = 0;
        for (RP k = rb + lane; k < re; k += kWave) {
          const int u = a.colidx[k];
          const int s = (u >= v0 && u < v1) ? a.color[u] : a.slot[k];
          const unsigned r = (unsigned)s - (unsigned)base;
          if (s >= 0 && r < 64u) m |= 1ull << r;
        }
        m = group_or<kWave>(m);
        if (m != ~0ull) {
          c = base + __builtin_ctzll(~m);
          break;
        }
      }
      if (lane == 0) a.color[v] = c;
      // later vertices of this block (same wavefront) read this colour
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    }
  }
}

// Phase 2 by 64-vertex chunks: the rows of a chunk's pending vertices are
// consecutive in colidx, so the wavefront streams them as one segmented
// list (coalesced reads of colidx, coalesced slot writes); entry j belongs to
// the last lane whose exclusive prefix is <= j (binary search over the
// prefixes with cross-lane reads), and the conflicts of the chunk meet in a
// 64-bit mask, bit i for lane i's vertex.
template <typename RP>
__global__ __launch_bounds__(kBlock) void k_blk_phase2(BArgs a) {
  __shared__ int sh_active, sh_lost;
  const RP* __restrict__ rp = (const RP*)a.rowptr;
  if (threadIdx.x == 0) {
    sh_active = 0;
    sh_lost = 0;
  }
  __syncthreads();
  int active = 0, lost = 0;
  const int lane = lane_id();
  const long wave_gid = blockIdx.x * (long)kWavesPerBlock + threadIdx.x / kWave;
  const long nwaves = (long)gridDim.x * kWavesPerBlock;
  const long nchunks = ((long)a.n + kWave - 1) / kWave;
  for (long ch = wave_gid; ch < nchunks; ch += nwaves) {
    const int v = (int)(ch * kWave) + lane;
    const bool pend = v < a.n && a.todo[v];
    RP b = 0;
    int len = 0, v0 = 0, v1 = 0, cv = 0;
    if (pend) {
      b = rp[v];
      len = (int)(rp[v + 1] - b);
      const long blk = (long)v * a.p / a.n;
      v0 = block_start(blk, a.n, a.p);
      v1 = block_start(blk + 1, a.n, a.p);
      cv = a.color[v];
    }
    if (__ballot(pend) == 0) continue;
    int incl = len;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int y = __shfl_up(incl, off);
      if (lane >= off) incl += y;
    }
    const int total = __shfl(incl, kWave - 1);
    const int excl = incl - len;
    uint64_t lm = 0;
    for (int j0 = 0; j0 < total; j0 += 4 * kWave) {
      int u[4], o[4], ov1[4], ocv[4];
      bool ok[4], foreign[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = j0 + q * kWave + lane;
        ok[q] = j < total;
        int lo = 0;
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) {
          const int mid = lo + w;
          const int pm = __shfl(excl, mid < kWave ? mid : kWave - 1);
          if (mid < kWave && pm <= j) lo = mid;
        }
        o[q] = lo;
        const RP ob = shfl_any<RP>(b, lo);
        const int oe = __shfl(excl, lo);
        const int ov0 = __shfl(v0, lo);
        ov1[q] = __shfl(v1, lo);
        ocv[q] = __shfl(cv, lo);
        u[q] = ok[q] ? a.colidx[ob + (j - oe)] : 0;
        foreign[q] = ok[q] && (u[q] < ov0 || u[q] >= ov1[q]);
        if (foreign[q]) {
          const int cu = a.color[u[q]];
          a.slot[ob + (j - oe)] = cu;
          if (cu == ocv[q] && u[q] >= ov1[q]) lm |= 1ull << o[q];  // higher block
        }
      }
    }
    lm = group_or<kWave>(lm);
    if (pend) {
      const bool lose = (lm >> lane) & 1;
      a.todo[v] = lose;
      active += 1;
      lost += lose;
    }
  }
  if (active) atomicAdd(&sh_active, active);
  if (lost) atomicAdd(&sh_lost, lost);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (sh_lost) atomicAdd(&a.ctrl->left.v, sh_lost);
    if (sh_active) {
      a.ctrl->last_round.v = a.round;
      if (a.round - 1 < kTraceRounds) atomicAdd(&a.ctrl->trace[a.round - 1], sh_active);
    }
  }
}

// ------------------------------------------------- masks for the slots --

// Blocks [x, y) of unit t are its vertices [block_start(x), block_start(y)).
struct UnitRange {
  int v0, v1;
};
__device__ __forceinline__ UnitRange unit_range(const BArgs& a, long t) {
  const long b0 = t * a.unit, b1 = min(b0 + a.unit, a.p);
  return {block_start(b0, a.n, a.p), block_start(b1, a.n, a.p)};
}

// Lanes of a group that reads a row, four entries per lane and step.
constexpr int kBlkLanes = 8;

// The rows of a chunk's marked lanes (am), a group of lanes each: f(pos,
// valid, u[4], ok[4]) per step of every group, done(pos, valid) per row, both in
// wave-uniform control flow; pos is the lane that owns the row.
template <typename RP, typename F, typename D>
__device__ __forceinline__ void chunk_rows(const int32_t* __restrict__ colidx, uint64_t am, RP b,
                                           RP e, F f, D done) {
  const int lane = lane_id();
  const int gl = lane & (kBlkLanes - 1);
  const int cnt = __popcll(am);
  const int from = pack_lanes(am, lane);
  for (int p = 0; p < cnt; p += kWave / kBlkLanes) {
    const int k = p + lane / kBlkLanes;
    const bool valid = k < cnt;
    const int pos = __shfl(from, k & (kWave - 1));
    RP i = shfl_any<RP>(b, pos) + gl;
    RP ve = shfl_any<RP>(e, pos);
    if (!valid) ve = i;
    while (__ballot(i < ve)) {
      int u[4];
      bool ok[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ok[j] = i + j * kBlkLanes < ve;
        u[j] = ok[j] ? colidx[i + j * kBlkLanes] : 0;
      }
      f(pos, valid, u, ok);
      i += 4 * kBlkLanes;
    }
    done(pos, valid);
  }
}

// Before round 1: no colour anywhere, every vertex to be coloured, and the
// neighbours in the own block as bits of the unit.
template <typename RP, int W>
__global__ __launch_bounds__(kBlock) void k_blkm_init(BArgs a) {
  const RP* __restrict__ rp = (const RP*)a.rowptr;
  const int lane = lane_id();
  const long wave_gid = blockIdx.x * (long)kWavesPerBlock + threadIdx.x / kWave;
  const long nwaves = (long)gridDim.x * kWavesPerBlock;
  const long nchunks = ((long)a.n + kWave - 1) / kWave;
  for (long ch = wave_gid; ch < nchunks; ch += nwaves) {
    const int v = (int)(ch * kWave) + lane;
    RP b = 0, e = 0;
    int v0 = 0, v1 = 0, u0 = 0;
    if (v < a.n) {
      b = rp[v];
      e = rp[v + 1];
      const long blk = (long)v * a.p / a.n;
      v0 = block_start(blk, a.n, a.p);
      v1 = block_start(blk + 1, a.n, a.p);
      u0 = unit_range(a, blk / a.unit).v0;
      a.st[v] = -1;
      a.todo[v] = 1;
      a.mask[2 * (long)v] = a.mask[2 * (long)v + 1] = 0;
    }
    uint64_t bits[W] = {};
    chunk_rows<RP>(
        a.colidx, __ballot(v < a.n), b, e,
        [&](int pos, bool, const int* u, const bool* ok) {
          const int ov0 = __shfl(v0, pos), ov1 = __shfl(v1, pos), ou0 = __shfl(u0, pos);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (ok[j] && u[j] >= ov0 && u[j] < ov1) {
              const int x = u[j] - ou0;
#pragma unroll
              for (int w = 0; w < W; ++w) bits[w] |= (x >> 6) == w ? 1ull << (x & 63) : 0;
            }
        },
        [&](int pos, bool valid) {
#pragma unroll
          for (int w = 0; w < W; ++w) {
            const uint64_t m = group_or<kBlkLanes>(bits[w]);
            bits[w] = 0;
            if (valid && (lane & (kBlkLanes - 1)) == 0)
              a.nb[(ch * kWave + pos) * W + w] = m;
          }
        });
  }
}

// Phase 1: one wavefront per unit of whole blocks (at most 64 W vertices).
template <int W>
__global__ __launch_bounds__(kBlock) void k_blkm_phase1(BArgs a) {
  if (blockIdx.x == 0) {
    fold_trace(a.ctrl, a.part);
    if (threadIdx.x == 0) a.ctrl->more[(a.round + 2) % 3].v = 0;
  }
  if (!a.ctrl->more[a.round % 3].v) return;
  const int lane = lane_id();
  const long wave_gid = blockIdx.x * (long)kWavesPerBlock + threadIdx.x / kWave;
  const long nwaves = (long)gridDim.x * kWavesPerBlock;
  const long units = (a.p + a.unit - 1) / a.unit;
  for (long t = wave_gid; t < units; t += nwaves) {
    const UnitRange r = unit_range(a, t);
    if (r.v0 >= r.v1) continue;
    int col[W];
    uint64_t lo[W], hi[W], nb[W][W], turn[W];
    bool pend[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const long v = (long)r.v0 + w * kWave + lane;
      col[w] = -1;
      lo[w] = hi[w] = 0;
      pend[w] = v < r.v1 && a.todo[v];
      if (v < r.v1) col[w] = a.st[v];
      uint64_t some = 0;
#pragma unroll
      for (int q = 0; q < W; ++q) nb[w][q] = 0;
      if (pend[w]) {
        lo[w] = a.mask[2 * v];
        hi[w] = a.mask[2 * v + 1];
#pragma unroll
        for (int q = 0; q < W; ++q) some |= nb[w][q] = a.nb[v * W + q];
      }
      // a vertex without neighbours in its block picks at once
      if (pend[w] && !some)
        col[w] = ~lo[w] ? __builtin_ctzll(~lo[w]) : 64 + __builtin_ctzll(~hi[w]);
      turn[w] = __ballot(pend[w] && some);
    }
    // the others in increasing id, the colours of the unit in registers
    auto lane64 = [](uint64_t x, int i) {
      return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), i) << 32) |
             (uint32_t)__builtin_amdgcn_readlane((int)x, i);
    };
    auto free_of = [](uint64_t l, uint64_t h) {
      return ~l ? __builtin_ctzll(~l) : 64 + __builtin_ctzll(~h);
    };
    if (a.round == 1) {
      // nothing is coloured before: each pick goes into the masks of its neighbours, one step
      // whatever their number (64 blocks of 157 vertices in cliques of 100: 1,036 us a call by
      // looking at each neighbour, 457 by slots, 286 now)
#pragma unroll
      for (int w = 0; w < W; ++w) {
        uint64_t m = turn[w];
        while (m) {  // wave-uniform
          const int i = __builtin_ctzll(m);
          m &= m - 1;
          const int c = free_of(lane64(lo[w], i), lane64(hi[w], i));
          if (lane == i) col[w] = c;
#pragma unroll
          for (int q = 0; q < W; ++q) {
            const bool near = (nb[q][w] >> i) & 1;
            lo[q] |= near && c < 64 ? 1ull << (c & 63) : 0;
            hi[q] |= near && c >= 64 ? 1ull << (c & 63) : 0;
          }
        }
      }
    } else {
#pragma unroll
      for (int w = 0; w < W; ++w) {
        uint64_t m = turn[w];
        while (m) {  // wave-uniform
          const int i = __builtin_ctzll(m);
          m &= m - 1;
          uint64_t l = lane64(lo[w], i), h = lane64(hi[w], i);
#pragma unroll
          for (int q = 0; q < W; ++q) {
            uint64_t b = lane64(nb[w][q], i);
            while (b) {
              const int j = __builtin_ctzll(b);
              b &= b - 1;
              const int c = __builtin_amdgcn_readlane(col[q], j);
              if (c >= 64) h |= 1ull << (c - 64);
              else if (c >= 0) l |= 1ull << c;
            }
          }
          const int c = free_of(l, h);
          if (lane == i) col[w] = c;
        }
      }
    }
#pragma unroll
    for (int w = 0; w < W; ++w)
      if (pend[w]) a.st[(long)r.v0 + w * kWave + lane] = (int8_t)col[w];
  }
}

// Phase 2: the colours of the neighbours in other blocks after this round's
// phase 1 decide who is recoloured, and are what phase 1 sees next.
template <typename RP>
__global__ __launch_bounds__(kBlock) void k_blkm_phase2(BArgs a) {
  __shared__ int sh_active[kWavesPerBlock], sh_lost[kWavesPerBlock];
  if (!a.ctrl->more[a.round % 3].v) return;
  const RP* __restrict__ rp = (const RP*)a.rowptr;
  const int8_t* __restrict__ st = a.st;
  int active = 0, lost = 0;
  const int lane = lane_id();
  const long wave_gid = blockIdx.x * (long)kWavesPerBlock + threadIdx.x / kWave;
  const long nwaves = (long)gridDim.x * kWavesPerBlock;
  const long nchunks = ((long)a.n + kWave - 1) / kWave;
  for (long ch = wave_gid; ch < nchunks; ch += nwaves) {
    const int v = (int)(ch * kWave) + lane;
    const bool pend = v < a.n && a.todo[v];
    const uint64_t am = __ballot(pend);
    if (am == 0) continue;
    RP b = 0, e = 0;
    int v0 = 0, v1 = 0, cv = 0;
    if (pend) {
      b = rp[v];
      e = rp[v + 1];
      const long blk = (long)v * a.p / a.n;
      v0 = block_start(blk, a.n, a.p);
      v1 = block_start(blk + 1, a.n, a.p);
      cv = st[v];
    }
    uint64_t lo = 0, hi = 0;
    bool hit = false;
    chunk_rows<RP>(
        a.colidx, am, b, e,
        [&](int pos, bool, const int* u, const bool* ok) {
          const int ov0 = __shfl(v0, pos), ov1 = __shfl(v1, pos), ocv = __shfl(cv, pos);
          int c[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) c[j] = ok[j] ? (int)st[u[j]] : -1;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const bool foreign = ok[j] && (u[j] < ov0 || u[j] >= ov1);
            const uint64_t bit = foreign ? 1ull << (c[j] & 63) : 0;
            lo |= c[j] < 64 ? bit : 0;
            hi |= c[j] < 64 ? 0 : bit;
            hit |= foreign && u[j] >= ov1 && c[j] == ocv;  // higher block
          }
        },
        [&](int pos, bool valid) {
          const uint64_t hm = __ballot(hit);
          const uint64_t gm = ((1ull << kBlkLanes) - 1) << (lane & ~(kBlkLanes - 1));
          const bool lose = valid && (hm & gm);
          if (hm) {
            const uint64_t l = group_or<kBlkLanes>(lo), h = group_or<kBlkLanes>(hi);
            if (lose && (lane & (kBlkLanes - 1)) == 0) {
              const long x = ch * kWave + pos;
              a.mask[2 * x] = l;
              a.mask[2 * x + 1] = h;
            }
          }
          if (valid && (lane & (kBlkLanes - 1)) == 0) {
            if (!lose) a.todo[ch * kWave + pos] = 0;
            active += 1;
            lost += lose;
          }
          lo = hi = 0;
          hit = false;
        });
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    active += __shfl_xor(active, off);
    lost += __shfl_xor(lost, off);
  }
  if (lane == 0) {
    sh_active[threadIdx.x / kWave] = active;
    sh_lost[threadIdx.x / kWave] = lost;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kWavesPerBlock; ++w) {
      active += sh_active[w];
      lost += sh_lost[w];
    }
    a.part[blockIdx.x] = active;
    if (lost && !a.ctrl->more[(a.round + 1) % 3].v) a.ctrl->more[(a.round + 1) % 3].v = 1;
    if (lost && a.count_left) atomicAdd(&a.ctrl->left.v, lost);
    if (blockIdx.x == 0) {
      a.ctrl->last_round.v = a.round;
      a.ctrl->pend.v = a.round;
      a.ctrl->pend_grid.v = (int)gridDim.x;
    }
  }
}

__global__ void k_blk_clear_left(Ctrl* c) {
  if (threadIdx.x == 0 && blockIdx.x == 0) c->left.v = 0;
}

template <typename RP>
static int launch_blocks_phase_t(const BArgs& a, int phase, int grid, hipStream_t s) {
  if (phase == 1) {
    hipLaunchKernelGGL(k_blk_clear_left, dim3(1), dim3(64), 0, s, a.ctrl);
    // enough wavefronts for one per block, capped by the grid of the round kernels
    const long waves = a.p;
    const int g1 = (int)std::min<long>((waves + kWavesPerBlock - 1) / kWavesPerBlock, (long)grid);
    hipLaunchKernelGGL((k_blk_phase1<RP>), dim3(std::max(1, g1)), dim3(kBlock), 0, s, a);
  } else {
    hipLaunchKernelGGL((k_blk_phase2<RP>), dim3(grid), dim3(kBlock), 0, s, a);
  }
  return (int)hipGetLastError();
}

__global__ void k_blk_set_left(Ctrl* c, int value) {
  if (threadIdx.x == 0 && blockIdx.x == 0) c->left.v = value;
}

int launch_blocks_set_left(Ctrl* c, int value, void* stream) {
  hipLaunchKernelGGL(k_blk_set_left, dim3(1), dim3(64), 0, (hipStream_t)stream, c, value);
  return (int)hipGetLastError();
}

int launch_blocks_init(const BArgs& a, bool rp64, int grid, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  if (rp64) hipLaunchKernelGGL((k_blk_init<int64_t>), dim3(grid), dim3(kBlock), 0, s, a);
  else hipLaunchKernelGGL((k_blk_init<int32_t>), dim3(grid), dim3(kBlock), 0, s, a);
  return (int)hipGetLastError();
}

#define GC_WORDS(KERNEL, ...)                                                                      \
  switch (a.words) {                                                                               \
    case 1: hipLaunchKernelGGL((KERNEL<__VA_ARGS__ 1>), dim3(grid), dim3(kBlock), 0, s, a); break; \
    case 2: hipLaunchKernelGGL((KERNEL<__VA_ARGS__ 2>), dim3(grid), dim3(kBlock), 0, s, a); break; \
    default: hipLaunchKernelGGL((KERNEL<__VA_ARGS__ 4>), dim3(grid), dim3(kBlock), 0, s, a);       \
  }

int launch_blkm_init(const BArgs& a, bool rp64, int grid, void* stream) {
  hipStream_t s = (hipStream_t)stream;
#define GC_RP32 int32_t,
#define GC_RP64 int64_t,
  if (rp64) {
    GC_WORDS(k_blkm_init, GC_RP64)
  } else {
    GC_WORDS(k_blkm_init, GC_RP32)
  }
  return (int)hipGetLastError();
}

int launch_blkm_phase(const BArgs& a, bool rp64, int phase, int grid, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  if (phase == 1) {
    GC_WORDS(k_blkm_phase1, )
  } else if (rp64) {
    hipLaunchKernelGGL((k_blkm_phase2<int64_t>), dim3(grid), dim3(kBlock), 0, s, a);
  } else {
    hipLaunchKernelGGL((k_blkm_phase2<int32_t>), dim3(grid), dim3(kBlock), 0, s, a);
  }
  return (int)hipGetLastError();
}

int launch_blocks_phase(const BArgs& a, bool rp64, int phase, int grid, void* stream) {
  return rp64 ? launch_blocks_phase_t<int64_t>(a, phase, grid, (hipStream_t)stream)
              : launch_blocks_phase_t<int32_t>(a, phase, grid, (hipStream_t)stream);
}

}  // namespace gc
