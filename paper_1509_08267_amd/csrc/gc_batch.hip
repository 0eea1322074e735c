// gc_batch.hip -- many independent graphs coloured in one launch.
//
// Each graph is coloured by one workgroup with exactly the rounds of the
// per-graph path (Algorithm 1 of Section 3.1 with every vertex its own
// block; the higher id of a conflicting pair is recoloured), so its colours
// are bit-identical to a gc_color call on it alone.  The batch only changes
// where the state lives and who runs it:
//   - a workgroup takes graphs from a device-side queue ordered largest
//     first (work buckets by log2 of the CSR size: longest-processing-time
//     order, so the big graphs do not finish last);
//   - a workgroup has a compute unit to itself and keeps the state of a graph
//     of up to 81,408 vertices (40,704 above a maximum degree of 127) in LDS
//     together with a mask of the colours taken at each vertex, which a
//     committing vertex marks in its neighbours (run_graph_push); the rows are
//     all that is left to read.  Other graphs gather their neighbours' states
//     every round, from LDS where the state alone fits there (int8 or int16 by
//     the maximum degree), else from an int32 state in the caller's colour array;
//   - a launch of many graphs that are nearly all small takes workgroups of a
//     quarter of the size, several to a compute unit (k_batch_small);
//   - the rounds are separated by workgroup barriers instead of grid-wide
//     ones, and each graph stops independently when its round has no loser;
//   - a graph that would outlast the rest of the launch (k_batch_plan) and has
//     work enough to occupy several workgroups is coloured by a team
//     of K workgroups instead: it appears K times in the queue, the K
//     workgroups that take those entries split its chunks, its rounds are
//     separated by a barrier of the team, and each member keeps a replica of
//     the state in LDS, reloaded from the shared colour array after every
//     barrier; so a large graph no longer holds the whole launch to one
//     workgroup's speed.
// The state between rounds is the colour array itself (final colours >= 0,
// ~t for a vertex still being coloured with tentative colour t) plus the
// round count, which makes a step of a few rounds resumable: gc_batch_step
// advances each listed graph by at most max_rounds rounds.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <type_traits>
#include <mutex>

#include "gc.h"
#include "gc_device.h"
#include "gc_internal.h"

namespace gc {

constexpr int kBatchBlock = 1024;         // threads per graph workgroup
constexpr int kBatchLds = 159 * 1024;     // LDS slice per workgroup (bytes): one per compute unit
constexpr int kBatchWaves = kBatchBlock / kWave;
#ifndef GC_BATCH_SPEC_QUADS
#define GC_BATCH_SPEC_QUADS 3
#endif
#ifndef GC_BATCH_ENTRIES_PER_LANE
#define GC_BATCH_ENTRIES_PER_LANE 12
#endif
#ifndef GC_BATCH_MIN_LANES
#define GC_BATCH_MIN_LANES 1
#endif
constexpr int kSpecQuads = GC_BATCH_SPEC_QUADS;  // row quads per lane in flight (speculate)
// lanes per vertex: the largest power of two from kMinLanes to 16 with at
// least kEntriesPerLane entries of an average row per lane
constexpr int kEntriesPerLane = GC_BATCH_ENTRIES_PER_LANE;
constexpr int kMinLanes = GC_BATCH_MIN_LANES;
constexpr int kBuckets = 64;
constexpr int kMaxTeams = 256;          // graphs coloured by a team, per launch
constexpr int kMaxExtraTickets = 4096;  // queue entries beyond one per graph
constexpr int64_t kMinTeamWork = 65536; // work (entries + vertices) per team member
// A member of a team works through kTeamCost times the work of a workgroup
// that has a graph to itself (the team gathers whole rows every round and
// meets at barriers, the other pushes into its own LDS), and a graph of
// at most kMinTeam work is done sooner alone than a team's barriers take.
constexpr uint64_t kTeamCost = 5;
constexpr uint64_t kMinTeam = 200000;
// Graphs that k_batch_small colours when there are many (see there).
constexpr int kSmallBlock = 256;
constexpr int kSmallMax = 4096;           // vertices at most
constexpr int kSmallBuckets = 16;         // work below 2^16
constexpr int kSmallLds = kSmallMax * 4;
constexpr int kSmallPerCu = 4;            // workgroups per CU (their registers)
constexpr int kFine = 512;  // work histogram of the plan: eight buckets per power of two
constexpr long kTeamSpinLimit = 1l << 25;

struct BatchCtrl {
  int32_t queue;    // next position in `order`
  int32_t tickets;  // entries of `order` for k_batch_color: one per graph, K per team graph
  int32_t small_queue;  // the same for k_batch_small, whose entries follow:
  int32_t small_end;    // [tickets, small_end)
  int32_t pad[60];
};

// Control words of one team (one 256-byte line each).
struct TeamCtrl {
  int32_t k;        // workgroups in the team
  int32_t joined;   // ranks handed out
  uint32_t arrive;  // barrier arrivals, counting up within the launch
  int32_t lost[3];  // "a vertex lost round r" at index r % 3
  int32_t left;     // vertices left uncoloured (summed over the team)
  int32_t maxdeg;   // maximum degree (over the team)
  int32_t abort;    // a barrier wait exceeded the spin limit
  int32_t pad[55];
};

// workspace: [BatchCtrl][teams: kMaxTeams TeamCtrl][order: T int32][slot: T int32]
//            [gk: G int32][descs: G gc_graph_desc (packed API only)], T = G + kMaxExtraTickets
__host__ __device__ constexpr size_t ws_teams_off() { return sizeof(BatchCtrl); }
__host__ __device__ constexpr size_t ws_order_off() {
  return ws_teams_off() + (size_t)kMaxTeams * sizeof(TeamCtrl);
}
__host__ __device__ constexpr size_t ws_slot_off(int64_t G) {
  return ws_order_off() + (size_t)(G + kMaxExtraTickets) * sizeof(int32_t);
}
__host__ __device__ constexpr size_t ws_gk_off(int64_t G) {
  return ws_slot_off(G) + (size_t)(G + kMaxExtraTickets) * sizeof(int32_t);
}
__host__ __device__ constexpr size_t ws_descs_off(int64_t G) {
  return (ws_gk_off(G) + (size_t)G * sizeof(int32_t) + 255) & ~(size_t)255;
}

// Descriptors of a packed batch.
__global__ void k_batch_descs(int64_t G, const int64_t* voff, const int64_t* eoff,
                              gc_graph_desc* d) {
  const long tid = blockIdx.x * (long)blockDim.x + threadIdx.x;
  const long nth = (long)gridDim.x * blockDim.x;
  for (long g = tid; g < G; g += nth) {
    gc_graph_desc x;
    x.rowptr_off = voff[g] + g;
    x.colidx_off = eoff[g];
    x.color_off = voff[g];
    x.n = (int32_t)(voff[g + 1] - voff[g]);
    x.rounds = 0;
    x.active = 0;
    x.max_degree = 0;
    d[g] = x;
  }
}

// Largest-first order and teams.  One workgroup buckets the graphs by
// floor(log2(work)) (batch_work) and writes them out bucket by bucket,
// largest bucket first.
//
// A graph that takes longer alone than the whole launch should would hold
// every other workgroup up at the end, so it gets a team.  With work in units
// of a workgroup's own pace, a launch of length T that colours the graphs of
// cost <= T alone and the others in teams costs
//   sum(cost <= T) + kTeamCost * sum(work of the others),
// and the T taken is the smallest one (of the histogram's bucket ends) that
// nwg workgroups can hold.  A graph of cost above T and work of at least
// kMinTeam is coloured by K = min(kTeamCost * work / T + 1, nwg / 2,
// work / kMinTeamWork) workgroups when K >= 2 and a team slot and K - 1 extra
// queue entries are left; its K entries are consecutive, with the team slot
// beside them (-1 for a graph of one workgroup).  Also resets the work queue.
// Measured, against a team of floor(2 work / fair share) from one fair share of
// the work up: 512 graphs of up to 50,000 vertices 2.19 ms (3.73), 100 graphs
// 1.05 (1.64), 12 graphs of up to 5,000 vertices 0.21 (0.44).
// The work of a graph: its CSR entries and vertices when fresh; when it
// resumes from an earlier step (rounds > 0), the vertices it left uncoloured
// times two more than its average degree, an estimate of what its next
// rounds visit, so that the order and the teams follow the work left.
__device__ __forceinline__ uint64_t batch_work(const gc_graph_desc& x, const int32_t* rowptr_base) {
  const int64_t nnz = x.n > 0 ? rowptr_base[x.rowptr_off + x.n] : 0;
  if (x.rounds > 0 && x.n > 0 && x.active >= 0 && x.active <= x.n)
    return (uint64_t)x.active * (uint64_t)(nnz / x.n + 2) + 1;
  return (uint64_t)nnz + (uint64_t)x.n + 1;
}

// What a graph costs a workgroup of its own: a graph beyond the masks of sixteen
// colours gathers, as a team would, or, up to 81,408 vertices, at least where its
// eight run out.
__device__ __forceinline__ uint64_t cost_alone(int n, uint64_t w) {
  return n > (kBatchLds - 4) / 3 ? kTeamCost * w : w;
}

// Bucket of x >= 1: its power of two and the next three bits.  The end of
// bucket b is the largest x in it, to within its eighth.
__device__ __forceinline__ int fine_bucket(uint64_t x) {
  const int p = 63 - __builtin_clzll(x);
  return min(kFine - 1, 8 * p + (p >= 3 ? (int)((x >> (p - 3)) & 7) : 0));
}
__device__ __forceinline__ uint64_t fine_end(int b) {
  return ((uint64_t)(9 + (b & 7)) << (b >> 3)) >> 3;
}

__device__ __forceinline__ bool is_small(int n, uint64_t w) {
  return n <= kSmallMax && w < (1ull << kSmallBuckets);
}
// Bucket of the order: below kSmallBuckets the graphs of k_batch_small, behind all others.
__device__ __forceinline__ int order_bucket(bool small, uint64_t w) {
  const int p = 63 - __builtin_clzll(w);
  return small ? p : min(kSmallBuckets + p, kBuckets - 1);
}

__global__ __launch_bounds__(1024) void k_batch_plan(int64_t G, const gc_graph_desc* d,
                                                     const int32_t* rowptr_base, int32_t* order,
                                                     int32_t* slot, int32_t* gk, TeamCtrl* teams,
                                                     BatchCtrl* ctrl, int nwg, int small) {
  __shared__ int hist[kBuckets];
  __shared__ int base[kBuckets];
  __shared__ unsigned long long alone[kFine], work[kFine];  // by cost alone
  __shared__ unsigned long long large;  // work of the graphs that are not small
  __shared__ int nteams, extra, len;
  for (int i = threadIdx.x; i < kBuckets; i += blockDim.x) hist[i] = 0;
  for (int i = threadIdx.x; i < kFine; i += blockDim.x) alone[i] = work[i] = 0;
  if (threadIdx.x == 0) {
    nteams = 0;
    extra = 0;
    large = 0;
    len = kFine - 1;
  }
  __syncthreads();
  uint64_t mine = 0;
  for (long g = threadIdx.x; g < G; g += blockDim.x) {
    const uint64_t w = batch_work(d[g], rowptr_base);
    const uint64_t c = cost_alone(d[g].n, w);
    const int b = fine_bucket(c);
    atomicAdd(&alone[b], (unsigned long long)c);
    atomicAdd(&work[b], (unsigned long long)w);
    mine += is_small(d[g].n, w) ? 0 : w;
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) mine += shfl_xor64(mine, off);
  if (lane_id() == 0 && mine) atomicAdd(&large, (unsigned long long)mine);
  __syncthreads();
  // prefix sums of `alone`, suffix sums of `work` (buckets above), in place
  const int b = threadIdx.x;
  for (int off = 1; off < kFine; off <<= 1) {
    unsigned long long x = 0, y = 0;
    if (b < kFine) {
      x = b >= off ? alone[b - off] : 0;
      y = b + off < kFine ? work[b + off] : 0;
    }
    __syncthreads();
    if (b < kFine) {
      alone[b] += x;
      work[b] += y;
    }
    __syncthreads();
  }
  if (b < 8 * 56) {  // (no batch reaches the buckets beyond)
    const uint64_t load = alone[b] + kTeamCost * work[b + 1];
    if (load <= (uint64_t)nwg * fine_end(b)) atomicMin(&len, b);
  }
  __syncthreads();
  const uint64_t T = fine_end(len);
  // k_batch_small runs after k_batch_color: only where that has next to nothing to do
  if (small) small = large <= work[0] / 64;
  for (long g = threadIdx.x; g < G; g += blockDim.x) {
    const uint64_t w = batch_work(d[g], rowptr_base);
    uint64_t q = 0;
    if (w >= kMinTeam && cost_alone(d[g].n, w) > T) {
      q = kTeamCost * w / T + 1;
      // half the units at most: a team waits for all its members, and another
      // kernel that needs its workgroups resident together may hold the rest
      if (q > (uint64_t)(nwg + 1) / 2) q = (uint64_t)(nwg + 1) / 2;
      if (q > w / kMinTeamWork) q = w / kMinTeamWork;
    }
    int k = 1, s = -1;
    if (q >= 2) {
      const int ts = atomicAdd(&nteams, 1);
      const int x = atomicAdd(&extra, (int)q - 1);
      if (ts < kMaxTeams && x + (int)q - 1 <= kMaxExtraTickets) {
        k = (int)q;
        s = ts;
        TeamCtrl* t = teams + s;
        t->k = k;
        t->joined = 0;
        t->arrive = 0;
        t->lost[0] = t->lost[1] = t->lost[2] = 0;
        t->left = 0;
        t->maxdeg = 0;
        t->abort = 0;
      }
    }
    gk[g] = k | ((s + 1) << 16);
    atomicAdd(&hist[order_bucket(small && is_small(d[g].n, w), w)], k);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int b = kBuckets - 1; b >= 0; --b) {
      base[b] = acc;
      acc += hist[b];
      if (b == kSmallBuckets) ctrl->tickets = acc;
    }
    ctrl->queue = ctrl->small_queue = 0;
    ctrl->small_end = acc;
  }
  __syncthreads();
  for (long g = threadIdx.x; g < G; g += blockDim.x) {
    const uint64_t w = batch_work(d[g], rowptr_base);
    const int k = gk[g] & 0xffff, s = (gk[g] >> 16) - 1;
    const int pos = atomicAdd(&base[order_bucket(small && is_small(d[g].n, w), w)], k);
    for (int j = 0; j < k; ++j) {
      order[pos + j] = (int32_t)g;
      slot[pos + j] = s;
    }
  }
}

struct GraphRun {
  const int32_t* rp;
  const int32_t* ci;
  int32_t* out;  // the graph's colour / state array (int32)
  int n;
  int rounds_in;
  int max_rounds;
};

// The row [b, e) read as aligned 16-byte quads: the quad holding entry b
// starts `lead` entries before it.  Every quad that holds at least one entry
// of the row lies inside the 16-byte block of an in-bounds entry, so it never
// leaves the array's last page; entries outside the row are masked.
struct Quads {
  const int4* q;
  int lead;  // entries of the first quad before b
  int len;   // lead + (e - b): entries from q[0] up to the row's end
};

__device__ __forceinline__ Quads quads_of(const int32_t* ci, int b, int e) {
  Quads r;
  r.lead = (int)(((uintptr_t)(ci + b) >> 2) & 3);
  r.q = (const int4*)(ci + b - r.lead);
  r.len = e - b + r.lead;
  return r;
}

__device__ __forceinline__ void unpack(const int4 w, int* u) {
  u[0] = w.x;
  u[1] = w.y;
  u[2] = w.z;
  u[3] = w.w;
}

// Least colour not final on any neighbour of the row [b, e), by a group of L
// lanes (gl = lane in group) with 16-byte loads, kSpecQuads quads per lane in
// flight.  Every lane returns the result.
template <typename State>
__device__ __forceinline__ int spec_quads(const int32_t* __restrict__ ci, const State& state,
                                          int b, int e, int L, int gl, int base0 = 0) {
  const Quads r = quads_of(ci, b, e);
  const int nq = (r.len + 3) >> 2;
  int base = base0;
  for (;;) {
    uint64_t m = 0;
    auto mark = [&](const int4 w, int idx0) {
      int u[4];
      unpack(w, u);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int idx = idx0 + j;
        if (idx >= r.lead && idx < r.len) {
          const int c = state(u[j]);
          const unsigned rel = (unsigned)c - (unsigned)base;
          if (c >= 0 && rel < 64u) m |= 1ull << rel;
        }
      }
    };
    for (int i = gl; i < nq; i += kSpecQuads * L) {
      // kSpecQuads quads per lane in flight, then their gathers
      int4 w[kSpecQuads];
#pragma unroll
      for (int j = 0; j < kSpecQuads; ++j)
        if (i + j * L < nq) w[j] = r.q[i + j * L];
#pragma unroll
      for (int j = 0; j < kSpecQuads; ++j)
        if (i + j * L < nq) mark(w[j], 4 * (i + j * L));
    }
    for (int off = L / 2; off > 0; off >>= 1) m |= shfl_xor64(m, off);
    if (m != ~0ull) return base + __builtin_ctzll(~m);
    base += 64;  // all of base..base+63 are taken: slide the window
  }
}

// Conflict scan of v (tentative colour t) over its lower neighbours, rows
// ascending, by a group of L lanes (lanes gbase .. gbase + L - 1, mask
// gmask) with 16-byte loads: each step covers L consecutive quads.  With
// `skip` (not null) the scan starts at offset *skip of the row, every lower
// neighbour before it being final, and leaves there the offset of the first
// lower neighbour seen still uncoloured, or of the point where the scan
// stopped when it saw none (the per-graph path's resume rule: final colours
// never change).  Stops at the first conflict or the first id >= v.
template <typename State>
__device__ __forceinline__ bool detect_quads(const int32_t* __restrict__ ci,
                                             const State& state, int b, int e, int v, int t,
                                             int L, int gl, uint64_t gmask, int gbase, int* skip) {
  const int from = skip ? *skip : 0;
  const Quads r = quads_of(ci, b + from, e);
  int first = -1;  // row offset of the first uncoloured lower neighbour seen
  for (int k0 = 0; k0 < r.len; k0 += 4 * L) {  // group-uniform
    const int k = k0 + 4 * gl;
    int u[4] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MAX};
    if (k < r.len) unpack(r.q[k >> 2], u);
    int ja = 4, jc = 4, jp = 4;  // this lane's first uncoloured / conflict / past entry
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int idx = k + j;
      if (idx < r.lead) continue;  // before the scan's start
      const bool in = idx < r.len;
      const bool low = in && u[j] < v;
      const int s = low ? state(u[j]) : 0;
      if (low && s < 0 && ja == 4) ja = j;
      // decode, do not test the sign: a neighbour that wins in this same
      // pass flips ~t to t concurrently and must still count
      if (low && tent_of(s) == t && jc == 4) jc = j;
      if (!low && jp == 4) jp = j;
    }
    const uint64_t am = (__ballot(ja < 4) & gmask) >> gbase;
    const uint64_t cm = (__ballot(jc < 4) & gmask) >> gbase;
    const uint64_t pm = (__ballot(jp < 4) & gmask) >> gbase;
    // offsets in the row of the first such entries (rows ascend, so every
    // lower entry precedes the first past one)
    auto pos = [&](uint64_t mask, int jl) {
      const int lane = __builtin_ctzll(mask);
      const int j = __shfl(jl, gbase + lane);
      return from + k0 + 4 * lane + j - r.lead;
    };
    if (first < 0 && am) first = pos(am, ja);
    if (cm) {
      if (skip) *skip = first >= 0 ? first : pos(cm, jc);
      return true;
    }
    if (pm) {
      if (skip) *skip = first >= 0 ? first : pos(pm, jp);
      return false;
    }
  }
  if (skip) *skip = first >= 0 ? first : e - b;
  return false;
}

// Lanes per item when cnt (>= 1) items share a wavefront: the largest power of
// two that gives every item a group at once.
__device__ __forceinline__ int group_lanes(int cnt) {
  return kWave >> (cnt <= 1 ? 0 : 32 - __builtin_clz((unsigned)cnt - 1));
}

// One pass (speculate or detect) of one round over the graph's uncoloured
// vertices by the whole workgroup (member `rank` of a team of K; 0 of 1
// alone): each wavefront walks 64-vertex chunks, ballots the uncoloured ones
// and hands them to its groups of L0 lanes, or of more when it has few of them
// (those left late are the ones with long rows: 600 R-MAT graphs of scale 17 that
// gather alone 1,372 -> 558 ms, 64 of scale 16 in teams 136 -> 46).  `skipv` (or null) holds each
// vertex's resume offset for the detect scans; `mirror` (or null) receives
// every state write as well (a team's shared copy).
template <typename S, bool SPEC>
__device__ __forceinline__ bool graph_pass(const GraphRun& g, S* st, int32_t* skipv, int L0,
                                           int rank = 0, int K = 1, int32_t* mirror = nullptr) {
  const int lane = lane_id();
  const int wave = threadIdx.x / kWave;
  const auto state = [st](int u) { return (int)st[u]; };
  bool lost = false;
  for (int ch = rank * kBatchWaves + wave; ch * kWave < g.n; ch += K * kBatchWaves) {
    const int v = ch * kWave + lane;
    bool act = false;
    int s = 0, b = 0, e = 0;
    if (v < g.n) {
      s = st[v];
      if (s < 0) {
        b = g.rp[v];
        e = g.rp[v + 1];
        act = true;
      }
    }
    const uint64_t am = __ballot(act);
    if (am == 0) continue;
    const int cnt = __popcll(am);
    const int L = max(L0, group_lanes(cnt));
    const int gl = lane & (L - 1);
    const int grp = lane / L;
    const uint64_t gmask = (L == kWave) ? ~0ull : (((1ull << L) - 1) << (grp * L));
    for (int p = 0; p < cnt; p += kWave / L) {
      const int k = p + grp;
      const bool valid = k < cnt;
      const int pos = nth_set_bit(am, valid ? k : 0);
      const int vb = __shfl(b, pos);
      const int ve = __shfl(e, pos);
      const int vs = __shfl(s, pos);
      const int vv = ch * kWave + pos;
      if (valid) {  // group-uniform
        if (SPEC) {
          const int t = spec_quads(g.ci, state, vb, ve, L, gl);
          if (gl == 0) {
            st[vv] = (S)~t;
            if (mirror) mirror[vv] = ~t;
          }
        } else {
          const int t = ~vs;
          int sk = skipv ? skipv[vv] : 0;
          const int sk0 = sk;
          const bool lose = detect_quads(g.ci, state, vb, ve, vv, t, L, gl, gmask, grp * L,
                                            skipv ? &sk : nullptr);
          if (gl == 0) {
            if (!lose) {
              st[vv] = (S)t;
              if (mirror) mirror[vv] = t;
            }
            if (skipv && sk != sk0) skipv[vv] = sk;
            lost |= lose;
          }
        }
      }
    }
  }
  return lost;
}

// Rounds of one graph until done or max_rounds more rounds have run.
// Returns the rounds completed; *left receives the vertices still uncoloured.
// A graph whose state is in LDS keeps each vertex's resume offset in its
// colour array during the rounds (the array receives the state at the end).
template <typename S, bool IN_LDS>
__device__ __forceinline__ int run_graph(const GraphRun& g, S* st, int L, int* left) {
  __shared__ int sh_cnt;
  int32_t* const skipv = IN_LDS ? g.out : nullptr;
  bool any = false;
  int r = g.rounds_in;
  if (r == 0) {
    // round 1 in closed form (sorted rows): v keeps colour 0 iff no neighbour
    // has a lower id
    for (int v = threadIdx.x; v < g.n; v += blockDim.x) {
      const int b = g.rp[v], e = g.rp[v + 1];
      const bool lose = e > b && g.ci[b] < v;
      st[v] = lose ? (S)-1 : (S)0;
      if (IN_LDS) skipv[v] = 0;
      any |= lose;
    }
    r = g.n > 0 ? 1 : 0;
  } else {
    for (int v = threadIdx.x; v < g.n; v += blockDim.x) {
      const int s = g.out[v];
      if (IN_LDS) {
        st[v] = (S)s;
        skipv[v] = 0;
      }
      any |= s < 0;
    }
  }
  bool more = __syncthreads_or(any);
  // (r < n: every round colours the lowest uncoloured vertex, so R <= n;
  // the bound only stops a broken invariant from spinning forever, and the
  // graph then reports uncoloured vertices)
  while (more && r < g.n && (g.max_rounds <= 0 || r - g.rounds_in < g.max_rounds)) {
    ++r;
    graph_pass<S, true>(g, st, skipv, L);
    __syncthreads();
    const bool lost = graph_pass<S, false>(g, st, skipv, L > 4 ? L / 2 : L);
    more = __syncthreads_or(lost);
  }
  if (threadIdx.x == 0) sh_cnt = 0;
  __syncthreads();
  int mine = 0;
  for (int v = threadIdx.x; v < g.n; v += blockDim.x) {
    const int s = st[v];
    if (IN_LDS) g.out[v] = s;
    mine += s < 0;
  }
  // (a cross-lane sum first: one LDS atomic per wave, not per thread)
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
  if (lane_id() == 0 && mine) atomicAdd(&sh_cnt, mine);
  __syncthreads();
  *left = sh_cnt;
  __syncthreads();
  return r;
}

// A graph's colouring state in the LDS slice under pushed colours: per
// vertex its state (~t or the final colour, in STATE bits: 8 up to a maximum
// degree of 127, 16 up to 32,767) and a mask of the colours below BITS that are
// final on a neighbour.  <24, 8> packs both into a word of 4 bytes, <16, 16> as
// well, <48, 16> into one of 8; <16, 8> takes 3 bytes and <8, 8> 2, two or four
// masks to a word before the states.
template <int BITS, int STATE>
struct Slots {
  using M = typename std::conditional<(BITS > 32), unsigned long long, uint32_t>::type;
  using S = typename std::conditional<STATE == 8, int8_t, int16_t>::type;
  static constexpr int kBits = BITS;
  static constexpr M kAll = ((M)1 << BITS) - 1;
  static constexpr bool kPacked = BITS + STATE == 8 * (int)sizeof(M);
  static constexpr int kStride = kPacked ? (int)(sizeof(M) / sizeof(S)) : 1;
  static constexpr int kPer = kPacked ? 1 : 32 / BITS;  // masks to a word
  M* w;
  S* st;
  __device__ static Slots at(char* smem, int n) {
    Slots x;
    x.w = (M*)smem;
    x.st = kPacked ? (S*)smem + kStride - 1 : (S*)(x.w + words(n));
    return x;
  }
  __device__ static constexpr int words(int n) { return (n + kPer - 1) / kPer; }
  __device__ static constexpr bool fits(int n) {
    return n <= kBatchLds && words(n) * (int)sizeof(M) + (kPacked ? 0 : n) <= kBatchLds;
  }
  __device__ static __forceinline__ int shift(int v) {
    return kPacked ? 0 : BITS * (int)((unsigned)v % kPer);
  }
  // state s and no mask (the split layout's masks are cleared apart)
  __device__ __forceinline__ void init(int v, int s) const {
    if (kPacked) w[v] = (M)(long long)s << (BITS & 63);
    else set_state(v, s);
  }
  __device__ __forceinline__ int state(int v) const { return st[kStride * v]; }
  __device__ __forceinline__ void set_state(int v, int s) const { st[kStride * v] = (S)s; }
  __device__ __forceinline__ M mask(int v) const {
    return (w[(unsigned)v / kPer] >> shift(v)) & kAll;
  }
  // several lanes may mark the vertices of one word
  __device__ __forceinline__ void mark(int v, M bits) const {
    atomicOr(&w[(unsigned)v / kPer], bits << shift(v));
  }
};

// A wavefront's vertices that have committed and not yet pushed: row segment
// [b, e) and colour t in lanes 0 .. cnt - 1.  They push together, a group of
// lanes each, so that few winners at a time still fill the wavefront.
template <typename SL>
struct Winners {
  int b = 0, e = 0, t = 0, cnt = 0;

  // marks the queued colours; four quads in flight per lane
  __device__ __forceinline__ void flush(const SL& sl, const int32_t* __restrict__ ci) {
    if (cnt == 0) return;
    const int lane = lane_id();
    const int L = min(16, group_lanes(cnt));
    const int gl = lane & (L - 1);
    for (int p = 0; p < cnt; p += kWave / L) {  // wave-uniform
      const int k = p + lane / L;
      const int vb = __shfl(b, k & (kWave - 1)), ve = __shfl(e, k & (kWave - 1)),
                vt = __shfl(t, k & (kWave - 1));
      if (k >= cnt) continue;
      const typename SL::M bit = (typename SL::M)1 << vt;
      const Quads r = quads_of(ci, vb, ve);
      const int nq = (r.len + 3) >> 2;
      for (int i = gl; i < nq; i += 4 * L) {
        int4 w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (i + j * L < nq) w[j] = r.q[i + j * L];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (i + j * L >= nq) break;
          int u[4];
          unpack(w[j], u);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int idx = 4 * (i + j * L) + q;
            if (idx >= r.lead && idx < r.len) sl.mark(u[q], bit);
          }
        }
      }
    }
    cnt = 0;
  }

  // the lanes of wm join the queue (all lanes active; colours with a mask bit)
  __device__ __forceinline__ void add(const SL& sl, const int32_t* __restrict__ ci, uint64_t wm,
                                      int pb, int pe, int pt) {
    const int c = __popcll(wm);
    if (c == 0) return;
    if (cnt + c > kWave) flush(sl, ci);
    const int qb = pack_lanes(wm, pb, cnt), qe = pack_lanes(wm, pe, cnt),
              qt = pack_lanes(wm, pt, cnt);
    if (lane_id() >= cnt) {
      b = qb;
      e = qe;
      t = qt;
    }
    cnt += c;
  }
};
constexpr int kPushBatch = 16;  // queued winners that are pushed at once

// Rounds of one graph by one workgroup with pushed colours, everything but the
// rows and the resume offsets in LDS: a vertex that commits marks its colour
// in its neighbours' masks (LDS atomics), so a speculate pass reads a word
// per uncoloured vertex and only a vertex with all colours below BITS taken
// scans its row.  Every row is then read about once for its pushes and in
// parts by the conflict scans, not whole in every round it stays uncoloured.
// Bound by the latency of the scans' row reads (about 230 M scattered 64-byte
// sectors per 4,096-graph batch, 16 wavefronts per unit to hide it) and, at
// 40% of the issue slots, by the instructions around them.  The batch, ms per
// launch: gathering every round 16.8; pushed masks with a chunk's scans and
// pushes in lockstep 10.9; uncoloured vertices packed across chunks 8.2; a new
// vertex for every lane that is done, winners pushing sixteen at a time 7.5.
template <typename SL, int WAVES = kBatchWaves>
__device__ __forceinline__ int run_graph_push(const GraphRun& g, char* smem, int L, int* left) {
  using M = typename SL::M;
  constexpr int BITS = SL::kBits;
  __shared__ int sh_cnt;
  const SL sl = SL::at(smem, g.n);
  const auto state = [sl](int u) { return sl.state(u); };
  int32_t* const skipv = g.out;  // the resume offsets, until the colours are written
  const int lane = lane_id();
  const int wave = threadIdx.x / kWave;
  const int gl = lane & (L - 1), grp = lane / L, Gw = kWave / L;
  const int nchunks = (g.n + kWave - 1) / kWave;
  bool any = false;
  int r = g.rounds_in;
  if (!SL::kPacked)
    for (int i = threadIdx.x; i < SL::words(g.n); i += blockDim.x) sl.w[i] = 0;
  for (int v = threadIdx.x; v < g.n; v += blockDim.x) {
    const int s = r == 0 ? -1 : g.out[v];
    sl.init(v, s);
    any |= s < 0;
  }
  __syncthreads();
  if (r == 0) {
    // round 1 in closed form (sorted rows): v keeps colour 0 iff no neighbour
    // has a lower id
    any = false;
    Winners<SL> wq;
    for (int ch = wave; ch < nchunks; ch += WAVES) {
      const int v = ch * kWave + lane;
      int b = 0, e = 0;
      bool win = false;
      if (v < g.n) {
        b = g.rp[v];
        e = g.rp[v + 1];
        win = e == b || g.ci[b] > v;
        if (win) sl.set_state(v, 0);
        skipv[v] = 0;
        any |= !win;
      }
      wq.add(sl, g.ci, __ballot(win && e > b), b, e, 0);
      if (wq.cnt >= kPushBatch) wq.flush(sl, g.ci);
    }
    wq.flush(sl, g.ci);
    r = g.n > 0 ? 1 : 0;
  } else {
    // resumed: the masks of the uncoloured vertices from their rows
    for (int ch = wave; ch < nchunks; ch += WAVES) {
      const int v = ch * kWave + lane;
      int b = 0, e = 0;
      bool act = false;
      if (v < g.n) {
        skipv[v] = 0;
        act = sl.state(v) < 0;
      }
      if (act) {
        b = g.rp[v];
        e = g.rp[v + 1];
      }
      const uint64_t am = __ballot(act);
      const int cnt = __popcll(am);
      for (int p = 0; p < cnt; p += Gw) {
        const int k = p + grp;
        const int pos = nth_set_bit(am, k < cnt ? k : 0);
        const int vb = __shfl(b, pos), ve = __shfl(e, pos);
        M m = 0;
        if (k < cnt) {
          const Quads q = quads_of(g.ci, vb, ve);
          for (int i = gl; 4 * i < q.len; i += L) {
            int u[4];
            unpack(q.q[i], u);
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (4 * i + j >= q.lead && 4 * i + j < q.len) {
                const int c = sl.state(u[j]);
                if (c >= 0 && c < BITS) m |= (M)1 << c;
              }
          }
        }
        for (int off = L / 2; off > 0; off >>= 1) m |= __shfl_xor(m, off);
        if (k < cnt && gl == 0 && m) sl.mark(ch * kWave + pos, m);
      }
    }
  }
  bool more = __syncthreads_or(any);
  // (r < n: every round colours the lowest uncoloured vertex, so R <= n;
  // the bound only stops a broken invariant from spinning forever, and the
  // graph then reports uncoloured vertices)
  while (more && r < g.n && (g.max_rounds <= 0 || r - g.rounds_in < g.max_rounds)) {
    ++r;
    for (int ch = wave; ch < nchunks; ch += WAVES) {  // speculate
      const int v = ch * kWave + lane;
      bool full = false;
      if (v < g.n && sl.state(v) < 0) {
        const M m = sl.mask(v);
        full = m == SL::kAll;
        if (!full) sl.set_state(v, ~__builtin_ctzll(~(unsigned long long)m));
      }
      const uint64_t fm = __ballot(full);
      if (fm == 0) continue;
      int b = 0, e = 0;
      if (full) {
        b = g.rp[v];
        e = g.rp[v + 1];
      }
      const int cnt = __popcll(fm);
      const int FL = max(L, group_lanes(cnt));  // few such rows are long ones
      for (int p = 0; p < cnt; p += kWave / FL) {
        const int k = p + lane / FL;
        const int pos = nth_set_bit(fm, k < cnt ? k : 0);
        const int vb = __shfl(b, pos), ve = __shfl(e, pos);
        if (k < cnt) {
          const int t = spec_quads(g.ci, state, vb, ve, FL, lane & (FL - 1), BITS);
          if ((lane & (FL - 1)) == 0) sl.set_state(ch * kWave + pos, ~t);
        }
      }
    }
    __syncthreads();
    // Detect, commit, push.  A wavefront packs the uncoloured vertices of its
    // chunks into batches of 64 whose row ends and offsets are loaded ahead.
    // Each lane scans a row, eight entries (two quads) a step, and takes the
    // next vertex of the batch as soon as its own is decided, so that every
    // step has 64 rows to read and a long scan holds up no other; the winners
    // push sixteen at a time while the next step's quads are on their way.
    bool lost = false;
    Winners<SL> wq;
    int ch = wave, pv = 0, pc = 0;  // next chunk; vertices packed so far, in lanes 0 .. pc - 1
    auto next_batch = [&](int& v) {
      while (ch < nchunks) {  // wave-uniform
        const int c0 = ch * kWave;
        ch += WAVES;
        const uint64_t am = __ballot(c0 + lane < g.n && sl.state(min(c0 + lane, g.n - 1)) < 0);
        const int total = pc + __popcll(am);
        if (total == pc) continue;
        const int q = pack_lanes(am, c0 + lane, pc);  // beyond lane 63 it wraps to lane 0
        if (lane >= pc) pv = q;
        pc = total;
        if (total < kWave) continue;
        v = pv;
        pv = q;
        pc = total - kWave;
        return kWave;
      }
      v = pv;
      const int c = pc;
      pc = 0;
      return c;
    };
    int qv = 0, qb = 0, qe = 0, qs = 0, qc = 0, qh = 0;  // the batch being handed out, its head
    int nv = 0, nb = 0, ne = 0, ns = 0;                  // the one after it
    auto load_next = [&]() {
      const int c = next_batch(nv);
      if (lane < c) {
        nb = g.rp[nv];
        ne = g.rp[nv + 1];
        ns = skipv[nv];
      }
      return c;
    };
    int nc = load_next();
    // this lane's scan: vertex v (-1: none), colour t, row [b, e); lo is where it
    // began, k the aligned entry of the step, first the first uncoloured lower
    // neighbour seen (-1: none); all but v and t are positions in colidx
    int v = -1, t = 0, b = 0, e = 0, lo = 0, k = 0, first = -1;
    // the scan of a lane ends at position `at`
    auto settle = [&](bool done, bool lose, int at) {
      const int sk = first >= 0 ? first : at;
      const bool win = done && !lose;
      if (win) sl.set_state(v, t);
      else if (done && sk != lo) skipv[v] = sk - b;
      lost |= done && lose;
      wq.add(sl, g.ci, __ballot(win && t < BITS && sk < e), sk, e, t);
      if (done) v = -1;
    };
    const int mis = (int)(((uintptr_t)g.ci >> 2) & 3);
    for (;;) {  // wave-uniform
      for (;;) {
        const uint64_t fm = __ballot(v < 0);
        if (fm == 0 || (qh == qc && nc == 0)) break;
        if (qh == qc) {
          qv = nv;
          qb = nb;
          qe = ne;
          qs = ns;
          qc = nc;
          qh = 0;
          nc = load_next();
        }
        const int take = min(__popcll(fm), qc - qh);
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(fm >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)fm, 0));
        const int from = (qh + rank) & (kWave - 1);
        const int xv = __shfl(qv, from), xb = __shfl(qb, from), xe = __shfl(qe, from),
                  xs = __shfl(qs, from);
        if (v < 0 && rank < take) {
          v = xv;
          b = xb;
          e = xe;
          lo = xb + xs;
          k = ((lo + mis) & ~3) - mis;
          first = -1;
          t = ~sl.state(v);
        }
        qh += take;
      }
      const uint64_t am = __ballot(v >= 0);
      const int cnt = __popcll(am);
      if (cnt == 0) break;
      if (cnt <= kSparseChunk) {  // (no vertex is left to hand out)
        // a group of lanes each for the rest
        const int GL = group_lanes(cnt);
        const int gi = lane / GL;
        const int pos = __shfl(pack_lanes(am, lane), gi);
        const int vv = __shfl(v, pos), vb = __shfl(b, pos), ve = __shfl(e, pos),
                  vt = __shfl(t, pos);
        int gsk = __shfl(max(k, lo) - b, pos), glose = 0;
        if (gi < cnt) {  // group-uniform
          const uint64_t gmask = GL == kWave ? ~0ull : ((1ull << GL) - 1) << (gi * GL);
          glose = detect_quads(g.ci, state, vb, ve, vv, vt, GL, lane & (GL - 1), gmask, gi * GL,
                               &gsk);
        }
        const int src = v >= 0 ? __popcll(am & ((1ull << lane) - 1)) * GL : 0;
        const int osk = __shfl(gsk, src), olose = __shfl(glose, src);
        settle(v >= 0, olose != 0, b + osk);
        break;
      }
      int4 wa = make_int4(0, 0, 0, 0), wb = wa;
      if (v >= 0) {
        if (k < e) wa = *(const int4*)(g.ci + k);
        if (k + 4 < e) wb = *(const int4*)(g.ci + k + 4);
      }
      if (wq.cnt >= kPushBatch) wq.flush(sl, g.ci);
      int u[8], s[8];
      unpack(wa, u);
      unpack(wb, u + 4);
      // An id of v or above ends the scan; such an entry (and one outside the
      // row, masked below) reads v's own state instead.
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j] = v >= 0 ? sl.state((int)min((unsigned)u[j], (unsigned)v)) : 0;
      uint32_t past = 0, hit = 0, open = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        past |= (uint32_t)((unsigned)u[j] >= (unsigned)v) << j;
        // decode, do not test the sign: a neighbour that wins in this same pass
        // flips ~t to t concurrently and must still count
        hit |= (uint32_t)(tent_of(s[j]) == t) << j;
        open |= (uint32_t)(s[j] < 0) << j;
      }
      past |= ~0u << min(max(e - k, 0), 8);
      const uint32_t seen = 0xffu & (~0u << min(max(lo - k, 0), 8));
      const uint32_t stop = (past | hit) & seen;
      const bool done = v >= 0 && stop != 0;
      const int at = stop ? __builtin_ctz(stop) : 8;
      const uint32_t before = open & seen & ((1u << at) - 1);
      if (first < 0 && before) first = k + __builtin_ctz(before);
      settle(done, !((past >> at) & 1), k + at);
      k += 8;
    }
    wq.flush(sl, g.ci);
    more = __syncthreads_or(lost);
  }
  if (threadIdx.x == 0) sh_cnt = 0;
  __syncthreads();
  int mine = 0;
  for (int v = threadIdx.x; v < g.n; v += blockDim.x) {
    const int s = sl.state(v);
    g.out[v] = s;
    mine += s < 0;
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
  if (lane_id() == 0 && mine) atomicAdd(&sh_cnt, mine);
  __syncthreads();
  *left = sh_cnt;
  __syncthreads();
  return r;
}

// Barrier of the K workgroups of a team.  Every member runs: each holds
// one of the team's K consecutive queue entries, a workgroup takes its next
// entry only after finishing its graph, and the graphs of earlier entries
// never wait on later ones, so the members of the earliest unfinished team
// are all taken (the launch is one workgroup per compute unit, all
// resident).  As the persistent kernel's grid barrier: agent-scope release
// and acquire around one arrival counter; a wait beyond the spin limit sets
// the team's abort flag, after which the team's barriers return at once.
__device__ __forceinline__ bool team_barrier(TeamCtrl* tc, int K, unsigned& phase) {
  __shared__ int sh_abort;
  drain_stores();
  __syncthreads();
  if (threadIdx.x == 0) {
    ++phase;
    const unsigned target = phase * (unsigned)K;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __hip_atomic_fetch_add(&tc->arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int ab = __hip_atomic_load(&tc->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    long spins = 0;
    while (!ab && __hip_atomic_load(&tc->arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
                      target) {
      __builtin_amdgcn_s_sleep(1);
      if (++spins > kTeamSpinLimit) {
        __hip_atomic_store(&tc->abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ab = 1;
      } else if ((spins & 1023) == 0) {
        ab = __hip_atomic_load(&tc->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    sh_abort = ab;
  }
  __syncthreads();
  return sh_abort == 0;
}

__device__ __forceinline__ int team_flag(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Start of a team's graph: each member takes every K-th vertex for round 1
// in closed form (or, on resumption, looks for vertices still uncoloured)
// and its share of the maximum degree; then the team's first barrier.  The
// shared state is the graph's colour array (int32).  "Some vertex lost round
// r" is gathered in tc->lost[r % 3]: set before the round's last barrier,
// read after it by every member (so all leave the loop together), and
// cleared by member 0 at the start of round r + 3, after every member has
// read it.
__device__ bool team_start(const GraphRun& g, TeamCtrl* tc, int rank, int K, unsigned& phase,
                           int& r) {
  int32_t* const st = g.out;
  const int t0 = rank * (int)blockDim.x + (int)threadIdx.x;
  const int tstride = K * (int)blockDim.x;
  bool any = false;
  int mx = 0;
  r = g.rounds_in;
  for (int v = t0; v < g.n; v += tstride) {
    const int b = g.rp[v], e = g.rp[v + 1];
    mx = max(mx, e - b);
    if (r == 0) {  // round 1 in closed form, as run_graph
      const bool lose = e > b && g.ci[b] < v;
      st[v] = lose ? -1 : 0;
      any |= lose;
    } else {
      any |= st[v] < 0;
    }
  }
  if (r == 0) r = g.n > 0 ? 1 : 0;
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) mx = max(mx, __shfl_xor(mx, off));
  if (lane_id() == 0 && mx) atomicMax(&tc->maxdeg, mx);
  if (__syncthreads_or(any) && threadIdx.x == 0) atomicOr(&tc->lost[r % 3], 1);
  return team_barrier(tc, K, phase);
}

// The rounds of one graph by member `rank` of a team of K workgroups: the
// same rounds as run_graph, each member taking every K-th 64-vertex chunk,
// the passes separated by team barriers.  With IN_LDS every member keeps a
// replica of the whole state in its LDS slice, reloaded from the shared
// colour array after each barrier, and writes its vertices to both, so the
// neighbour gathers stay LDS reads; otherwise the passes work on the shared
// array.  Returns the rounds completed; *left receives the vertices still
// uncoloured (all of them if a barrier gave up).
template <typename S, bool IN_LDS>
__device__ int team_rounds(const GraphRun& g, S* lds, TeamCtrl* tc, int rank, int K, int L,
                           unsigned& phase, int r, bool ok, int* left) {
  __shared__ int sh_cnt;
  int32_t* const gst = g.out;
  S* const st = IN_LDS ? lds : (S*)gst;
  int32_t* const mirror = IN_LDS ? gst : nullptr;
  // the shared array read as aligned 16-byte quads (as quads_of: every quad
  // read holds at least one of the graph's entries), four per thread in flight
  const int lead = (int)(((uintptr_t)gst >> 2) & 3);
  const int4* const q = (const int4*)(gst - lead);
  const int nq = (g.n + lead + 3) >> 2;
  auto reload = [&]() {
    if (IN_LDS) {
      for (int i0 = threadIdx.x; i0 < nq; i0 += 4 * blockDim.x) {
        int4 w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (i0 + j * (int)blockDim.x < nq) w[j] = q[i0 + j * blockDim.x];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int i = i0 + j * (int)blockDim.x;
          if (i >= nq) continue;
          int u[4];
          unpack(w[j], u);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int v = 4 * i + k - lead;
            if (v >= 0 && v < g.n) lds[v] = (S)u[k];
          }
        }
      }
      __syncthreads();
    }
  };
  bool more = ok && team_flag(&tc->lost[r % 3]) != 0;
  while (more && r < g.n && (g.max_rounds <= 0 || r - g.rounds_in < g.max_rounds)) {
    ++r;
    if (rank == 0 && threadIdx.x == 0)
      __hip_atomic_store(&tc->lost[r % 3], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    reload();
    graph_pass<S, true>(g, st, nullptr, L, rank, K, mirror);
    if (!(ok = team_barrier(tc, K, phase))) break;
    reload();
    const bool lost = graph_pass<S, false>(g, st, nullptr, L > 4 ? L / 2 : L, rank, K, mirror);
    if (__syncthreads_or(lost) && threadIdx.x == 0) atomicOr(&tc->lost[r % 3], 1);
    if (!(ok = team_barrier(tc, K, phase))) break;
    more = team_flag(&tc->lost[r % 3]) != 0;
  }
  int mine = 0;
  for (int v = rank * (int)blockDim.x + (int)threadIdx.x; v < g.n; v += K * (int)blockDim.x)
    mine += gst[v] < 0;
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
  if (threadIdx.x == 0) sh_cnt = 0;
  __syncthreads();
  if (lane_id() == 0 && mine) atomicAdd(&sh_cnt, mine);
  __syncthreads();
  if (threadIdx.x == 0 && sh_cnt) atomicAdd(&tc->left, sh_cnt);
  ok = team_barrier(tc, K, phase) && ok;
  *left = ok ? team_flag(&tc->left) : g.n;
  return r;
}

// A team member's whole graph: the start, then the rounds with the state
// placement run_graph would pick (by the team's maximum degree).
__device__ __forceinline__ int run_team(const GraphRun& g, char* smem, TeamCtrl* tc, int rank, int K, int L,
                        int* left) {
  unsigned phase = 0;
  int r = 0;
  const bool ok = team_start(g, tc, rank, K, phase, r);
  const int maxdeg = team_flag(&tc->maxdeg);  // complete: every member added it before the barrier
  if (maxdeg <= 127 && g.n <= kBatchLds)
    return team_rounds<int8_t, true>(g, (int8_t*)smem, tc, rank, K, L, phase, r, ok, left);
  if (maxdeg <= 32767 && 2 * g.n <= kBatchLds)
    return team_rounds<int16_t, true>(g, (int16_t*)smem, tc, rank, K, L, phase, r, ok, left);
  return team_rounds<int32_t, false>(g, nullptr, tc, rank, K, L, phase, r, ok, left);
}

// The widest masks that fit the slice beside the state (8 bits up to a maximum degree of 127, 16 up
// to 32,767); a state without masks where none do, and the caller's array where that does not fit.
// With a workgroup to a compute unit a graph that gathers alone has half the wavefronts it had with
// two, so the masks reach as far as they can.  ms per launch, gathering by two workgroups per unit /
// by one / with masks: 512 R-MAT graphs of scale 12 and edge factor 8 4.39 / 7.79 / 0.72, of scale
// 14 61.3 / 66.5 / 2.9, 64 of scale 15 and edge factor 16 46.3 / 123 / 30, 512 graphs of 2,000
// vertices and average degree 300 11.2 / 15.5 / 4.7, 600 of 60,000 and 16 9.38 / 11.3 / 4.5.
__device__ __forceinline__ int dispatch_state(const GraphRun& g, int maxdeg, char* smem, int L,
                                              int* left) {
  if (maxdeg <= 127 && Slots<24, 8>::fits(g.n))
    return run_graph_push<Slots<24, 8>>(g, smem, L, left);
  if (maxdeg <= 127 && Slots<16, 8>::fits(g.n))
    return run_graph_push<Slots<16, 8>>(g, smem, L, left);
  if (maxdeg <= 127 && Slots<8, 8>::fits(g.n)) return run_graph_push<Slots<8, 8>>(g, smem, L, left);
  if (maxdeg <= 32767 && Slots<48, 16>::fits(g.n))
    return run_graph_push<Slots<48, 16>>(g, smem, L, left);
  if (maxdeg <= 32767 && Slots<16, 16>::fits(g.n))
    return run_graph_push<Slots<16, 16>>(g, smem, L, left);
  if (maxdeg <= 127 && g.n <= kBatchLds) return run_graph<int8_t, true>(g, (int8_t*)smem, L, left);
  if (maxdeg <= 32767 && 2 * g.n <= kBatchLds)
    return run_graph<int16_t, true>(g, (int16_t*)smem, L, left);
  return run_graph<int32_t, false>(g, g.out, L, left);
}

// The maximum degree of a graph (workgroup-wide; *sh starts at 0) and the lanes per row.
__device__ __forceinline__ int graph_degrees(const GraphRun& g, int* sh, int* lanes) {
  int mx = 0;
  for (int v = threadIdx.x; v < g.n; v += blockDim.x) mx = max(mx, g.rp[v + 1] - g.rp[v]);
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) mx = max(mx, __shfl_xor(mx, off));
  if (lane_id() == 0 && mx) atomicMax(sh, mx);
  __syncthreads();
  const double avg = g.n > 0 ? (double)g.rp[g.n] / g.n : 0.0;
  int L = kMinLanes;
  while (L < 16 && 2.0 * L * kEntriesPerLane <= avg) L *= 2;
  *lanes = L;
  return *sh;
}

__global__ __launch_bounds__(kBatchBlock, 4) void k_batch_color(gc_graph_desc* d,
                                                            const int32_t* rowptr_base,
                                                            const int32_t* colidx_base,
                                                            int32_t* colors_base, int max_rounds,
                                                            const int32_t* order,
                                                            const int32_t* slot, TeamCtrl* teams,
                                                            BatchCtrl* ctrl) {
  extern __shared__ char smem[];
  __shared__ int sh_idx, sh_max, sh_rank;
  const int tickets = ctrl->tickets;
  for (;;) {
    if (threadIdx.x == 0) {
      sh_idx = atomicAdd(&ctrl->queue, 1);
      sh_max = 0;
    }
    __syncthreads();
    const int idx = sh_idx;
    if (idx >= tickets) break;  // workgroup-uniform
    const int gi = order[idx];
    const int ts = slot[idx];
    const gc_graph_desc x = d[gi];
    GraphRun g;
    g.rp = rowptr_base + x.rowptr_off;
    g.ci = colidx_base + x.colidx_off;
    g.out = colors_base + x.color_off;
    g.n = x.n;
    g.rounds_in = x.rounds;
    g.max_rounds = max_rounds;
    if (ts >= 0) {  // one member of a team (workgroup-uniform)
      TeamCtrl* tc = teams + ts;
      if (threadIdx.x == 0) sh_rank = atomicAdd(&tc->joined, 1);
      __syncthreads();
      const int rank = sh_rank, K = tc->k;
      const double avg = g.n > 0 ? (double)g.rp[g.n] / g.n : 0.0;
      int L = kMinLanes;
      while (L < 16 && 2.0 * L * kEntriesPerLane <= avg) L *= 2;
      int left = 0;
      const int rounds = run_team(g, smem, tc, rank, K, L, &left);
      if (rank == 0 && threadIdx.x == 0) {
        d[gi].rounds = rounds;
        d[gi].active = left;
        d[gi].max_degree = team_flag(&tc->maxdeg);
      }
      __syncthreads();  // sh_idx / sh_rank are rewritten for the next entry
      continue;
    }
    int left = 0, L = 0;
    const int maxdeg = graph_degrees(g, &sh_max, &L);
    const int rounds = dispatch_state(g, maxdeg, smem, L, &left);
    if (threadIdx.x == 0) {
      d[gi].rounds = rounds;
      d[gi].active = left;
      d[gi].max_degree = maxdeg;
    }
    __syncthreads();  // sh_idx / sh_max are rewritten for the next graph
  }
}

// Many small graphs (a launch of at least kSmallPerCu graphs per compute unit, nearly all of its
// work in graphs of up to kSmallMax vertices): workgroups of four wavefronts, several to a
// compute unit.  A small graph keeps few wavefronts busy and is bound by the chain of loads and
// barriers of its rounds, so what counts is how many are in flight, where a large one wants the
// LDS of a compute unit to itself.  20,000 graphs of 100 vertices: 1.73 ms by one workgroup per
// unit, 1.35 by two of half the LDS, now 0.61; 4,096 of 500: 0.52, 0.46, 0.25.  Beside large graphs
// the two kernels, one after the other, lose: 1,500 graphs of 100 to 50,000 vertices 1.43 ms
// against 1.28, 3,000 of 1,000 and two of 300,000 1.22 against 1.15.
__global__ __launch_bounds__(kSmallBlock, kSmallPerCu) void k_batch_small(
    gc_graph_desc* d, const int32_t* rowptr_base, const int32_t* colidx_base, int32_t* colors_base,
    int max_rounds, const int32_t* order, BatchCtrl* ctrl) {
  extern __shared__ char smem[];
  __shared__ int sh_idx, sh_max;
  constexpr int kWaves = kSmallBlock / kWave;
  const int first = ctrl->tickets, end = ctrl->small_end;
  for (;;) {
    if (threadIdx.x == 0) {
      sh_idx = first + atomicAdd(&ctrl->small_queue, 1);
      sh_max = 0;
    }
    __syncthreads();
    const int idx = sh_idx;
    if (idx >= end) break;  // workgroup-uniform
    const int gi = order[idx];
    const gc_graph_desc x = d[gi];
    GraphRun g;
    g.rp = rowptr_base + x.rowptr_off;
    g.ci = colidx_base + x.colidx_off;
    g.out = colors_base + x.color_off;
    g.n = x.n;
    g.rounds_in = x.rounds;
    g.max_rounds = max_rounds;
    int left = 0, L = 0;
    const int maxdeg = graph_degrees(g, &sh_max, &L);
    const int rounds = maxdeg <= 127 ? run_graph_push<Slots<24, 8>, kWaves>(g, smem, L, &left)
                                     : run_graph_push<Slots<16, 16>, kWaves>(g, smem, L, &left);
    if (threadIdx.x == 0) {
      d[gi].rounds = rounds;
      d[gi].active = left;
      d[gi].max_degree = maxdeg;
    }
    __syncthreads();  // sh_idx / sh_max are rewritten for the next graph
  }
}

__global__ void k_batch_rounds_out(int64_t G, const gc_graph_desc* d, int32_t* rounds_out) {
  const long tid = blockIdx.x * (long)blockDim.x + threadIdx.x;
  const long nth = (long)gridDim.x * blockDim.x;
  for (long g = tid; g < G; g += nth) rounds_out[g] = d[g].rounds;
}

static int batch_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 1;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) cus = 1;
  return cus > 0 ? cus : 1;
}

static int run_batch(int64_t G, gc_graph_desc* d, const int32_t* rpb, const int32_t* cib,
                     int32_t* colb, int max_rounds, void* ws, hipStream_t s) {
  const int rc = allow_lds((const void*)k_batch_color, kBatchLds);
  if (rc) return rc;
  BatchCtrl* ctrl = (BatchCtrl*)ws;
  TeamCtrl* teams = (TeamCtrl*)((char*)ws + ws_teams_off());
  int32_t* order = (int32_t*)((char*)ws + ws_order_off());
  int32_t* slot = (int32_t*)((char*)ws + ws_slot_off(G));
  int32_t* gk = (int32_t*)((char*)ws + ws_gk_off(G));
  // one workgroup per compute unit, all resident at once, whatever the number
  // of graphs: a team can use workgroups beyond one per graph
  const int grid = batch_cus();
  const bool small = G >= (int64_t)kSmallPerCu * grid;
  hipLaunchKernelGGL(k_batch_plan, dim3(1), dim3(1024), 0, s, G, d, rpb, order, slot, gk, teams,
                     ctrl, grid, (int)small);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return (int)e;
  hipLaunchKernelGGL(k_batch_color, dim3(grid), dim3(kBatchBlock), kBatchLds, s, d, rpb, cib, colb,
                     max_rounds, order, slot, teams, ctrl);
  e = hipGetLastError();
  if (e != hipSuccess || !small) return (int)e;
  hipLaunchKernelGGL(k_batch_small, dim3(kSmallPerCu * grid), dim3(kSmallBlock), kSmallLds, s, d,
                     rpb, cib, colb, max_rounds, order, ctrl);
  return (int)hipGetLastError();
}

}  // namespace gc

using namespace gc;

namespace {
int fail(int code, const char* msg) {
  set_thread_error(msg);
  return code;
}
}  // namespace

extern "C" size_t gc_batch_workspace_bytes(int64_t num_graphs, const int64_t* voff,
                                           const int64_t* eoff) {
  if (num_graphs < 0 || num_graphs > INT32_MAX || !voff || !eoff) return 0;
  if (voff[0] != 0 || eoff[0] != 0) return 0;
  for (int64_t g = 0; g < num_graphs; ++g) {
    const int64_t n = voff[g + 1] - voff[g], nnz = eoff[g + 1] - eoff[g];
    if (n < 0 || nnz < 0 || n >= INT32_MAX || nnz > INT32_MAX) return 0;
  }
  return ws_descs_off(num_graphs) + (size_t)num_graphs * sizeof(gc_graph_desc) + 256;
}

extern "C" int gc_color_batch(int64_t num_graphs, const int64_t* voff, const int64_t* eoff,
                              const int32_t* rowptr_local, const int32_t* colidx_local,
                              int32_t* colors_out, int32_t* rounds_out, void* workspace,
                              size_t workspace_bytes, void* stream) {
  if (num_graphs < 0 || num_graphs > INT32_MAX) return fail(GC_EINVAL, "gc_color_batch: bad num_graphs");
  if (num_graphs == 0) return GC_OK;
  if (!voff || !eoff || !rowptr_local || !workspace)
    return fail(GC_EINVAL, "gc_color_batch: NULL array");
  const size_t need = ws_descs_off(num_graphs) + (size_t)num_graphs * sizeof(gc_graph_desc) + 256;
  if (workspace_bytes < need) return fail(GC_EINVAL, "gc_color_batch: workspace too small");
  hipStream_t s = (hipStream_t)stream;
  (void)hipGetLastError();
  gc_graph_desc* d = (gc_graph_desc*)((char*)workspace + ws_descs_off(num_graphs));
  const int grid = (int)((num_graphs + 255) / 256 < 4096 ? (num_graphs + 255) / 256 : 4096);
  hipLaunchKernelGGL(k_batch_descs, dim3(grid), dim3(256), 0, s, num_graphs, voff, eoff, d);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(GC_EDEVICE, hipGetErrorString(e));
  int rc = run_batch(num_graphs, d, rowptr_local, colidx_local, colors_out, 0, workspace, s);
  if (rc) return fail(GC_EDEVICE, hipGetErrorString((hipError_t)rc));
  if (rounds_out) {
    hipLaunchKernelGGL(k_batch_rounds_out, dim3(grid), dim3(256), 0, s, num_graphs, d, rounds_out);
    e = hipGetLastError();
    if (e != hipSuccess) return fail(GC_EDEVICE, hipGetErrorString(e));
  }
  return GC_OK;
}

// ------------------------------------------ batch without allocation --

namespace gc {

// Workspace of gc_color_batch_noalloc: a file-scope device array of
// kStaticBatchBytes, enough for kStaticBatchGraphs graphs.  Each GPU holds
// its own copy from the first launch of this library's kernels on it until
// the process ends.
constexpr int64_t kStaticBatchGraphs = GC_STATIC_BATCH_MAX_GRAPHS;
constexpr size_t kStaticBatchBytes =
    ws_descs_off(kStaticBatchGraphs) + (size_t)kStaticBatchGraphs * sizeof(gc_graph_desc) + 256;
static __device__ __align__(256) uint8_t scratch[kStaticBatchBytes];

// Device address of `scratch` on each device, looked up once per device with
// that device current (host code never passes the array's name itself).
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kMaxDevices] = {};

static int static_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    if (!p) return (int)hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return 0;
}

}  // namespace gc

extern "C" int gc_color_batch_noalloc(int64_t num_graphs, const int64_t* voff, const int64_t* eoff,
                                      const int32_t* rowptr_local, const int32_t* colidx_local,
                                      int32_t* colors_out, int32_t* rounds_out, void* stream) {
  if (num_graphs < 0) return fail(GC_EINVAL, "gc_color_batch_noalloc: bad num_graphs");
  if (num_graphs > gc::kStaticBatchGraphs)
    return fail(GC_ETOOBIG, "gc_color_batch_noalloc: more graphs than GC_STATIC_BATCH_MAX_GRAPHS");
  if (num_graphs == 0) return GC_OK;
  void* ws = nullptr;
  const int rc = gc::static_scratch(&ws);
  if (rc) return fail(GC_EDEVICE, hipGetErrorString((hipError_t)rc));
  return gc_color_batch(num_graphs, voff, eoff, rowptr_local, colidx_local, colors_out,
                        rounds_out, ws, gc::kStaticBatchBytes, stream);
}

extern "C" size_t gc_batch_step_workspace_bytes(int64_t num_graphs, int64_t total_vertices) {
  if (num_graphs < 0 || num_graphs > INT32_MAX || total_vertices < 0) return 0;
  return ws_descs_off(num_graphs) + 256;
}

extern "C" int gc_batch_step(int64_t num_graphs, gc_graph_desc* descs, const int32_t* rowptr_base,
                             const int32_t* colidx_base, int32_t* colors_base, int32_t max_rounds,
                             void* workspace, size_t workspace_bytes, void* stream) {
  if (num_graphs < 0 || num_graphs > INT32_MAX) return fail(GC_EINVAL, "gc_batch_step: bad num_graphs");
  if (num_graphs == 0) return GC_OK;
  if (!descs || !rowptr_base || !workspace) return fail(GC_EINVAL, "gc_batch_step: NULL array");
  if (max_rounds < 0) return fail(GC_EINVAL, "gc_batch_step: negative max_rounds");
  if (workspace_bytes < gc_batch_step_workspace_bytes(num_graphs, 0))
    return fail(GC_EINVAL, "gc_batch_step: workspace too small");
  (void)hipGetLastError();
  int rc = run_batch(num_graphs, descs, rowptr_base, colidx_base, colors_base, max_rounds,
                     workspace, (hipStream_t)stream);
  if (rc) return fail(GC_EDEVICE, hipGetErrorString((hipError_t)rc));
  return GC_OK;
}

// ------------------------------------------------- segment copies --

namespace gc {

// Piece p of the concatenated segments: the segment is the last one whose
// first piece is <= p (binary search, the same in every thread of the
// workgroup), and the piece covers words [q * P, min((q + 1) * P, words)) of
// it, q = p - first_piece.
__global__ __launch_bounds__(kBlock) void k_copy_segments(const gc_segment* __restrict__ seg,
                                                          int64_t count, int64_t pieces) {
  for (int64_t p = blockIdx.x; p < pieces; p += gridDim.x) {  // workgroup-uniform
    int64_t lo = 0, hi = count - 1;
    while (lo < hi) {
      const int64_t mid = lo + (hi - lo + 1) / 2;
      if (seg[mid].first_piece <= p) lo = mid;
      else hi = mid - 1;
    }
    const gc_segment x = seg[lo];
    const int64_t start = (p - x.first_piece) * GC_COPY_PIECE_WORDS;
    if (start < 0 || start >= x.words) continue;
    const int64_t end = start + GC_COPY_PIECE_WORDS < x.words ? start + GC_COPY_PIECE_WORDS : x.words;
    const int32_t* __restrict__ src = (const int32_t*)x.src;
    int32_t* __restrict__ dst = (int32_t*)x.dst;
    for (int64_t k = start + threadIdx.x; k < end; k += blockDim.x) dst[k] = src[k];
  }
}

}  // namespace gc

extern "C" int gc_copy_segments(int64_t count, const gc_segment* segs, int64_t pieces,
                                void* stream) {
  if (count < 0 || pieces < 0) return fail(GC_EINVAL, "gc_copy_segments: negative count or pieces");
  if (count == 0 || pieces == 0) return GC_OK;
  if (!segs) return fail(GC_EINVAL, "gc_copy_segments: NULL descriptors");
  (void)hipGetLastError();
  const int grid = (int)(pieces < 4096 ? pieces : 4096);
  hipLaunchKernelGGL(gc::k_copy_segments, dim3(grid), dim3(gc::kBlock), 0, (hipStream_t)stream,
                     segs, count, pieces);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(GC_EDEVICE, hipGetErrorString(e));
  return GC_OK;
}

