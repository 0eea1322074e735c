// gc_resident.hip -- a whole colouring in one launch, the graph resident in LDS.
//
// A graph of some ten thousand vertices is bound by its rounds' launches and
// dependent loads (two passes, 12 us a round), not by its work.  Up to
// kResGroups workgroups share it: the 64-vertex chunks are dealt round-robin,
// a workgroup copies the rows of its chunks into LDS once (16-bit neighbour ids)
// and keeps a replica of every vertex's one-byte state.  A round is then
//   detect      each own uncoloured vertex against the replica; winners are
//               published, 32 vertices to a word, and everybody's read;
//   speculate   each own vertex still uncoloured takes the least colour not
//               final in its row; the states are published, six to a word, and
//               everybody's read.
// Round 1 starts with detect: every vertex tries colour 0.  Every published
// word carries its round, so that a reader polls the data itself.  Words
// without an uncoloured vertex are neither published nor read (all replicas
// agree on what is final).  A workgroup whose last vertices win leaves as soon
// as it has published them, and reads nothing more: nobody waits for it from
// then on, so a word that it still meant to read could be overwritten by the
// next round's.  Everybody who reads the winners has vertices left and
// publishes their states afterwards, and everybody who reads the states
// publishes winners afterwards, so a word is rewritten only after all its
// readers have read it: one buffer of each suffices.
//
// Bound by the two exchanges and the workgroup barriers around them, 7 us a
// round.  Whole calls, uniform random graphs, before and after: 4,000 vertices
// of average degree 24 198 -> 117 us, 10,000 of 20 181 -> 120, 16,000 of 8
// 115 -> 94, 20,000 of 30 255 -> 188; at 30,000 of 20 both take 190 and at
// 40,000 of 8 the rounds' own passes are ahead (116 against 140), as every
// workgroup reads every vertex's state, so the pass ends at 24,576 vertices.
//
// As in the core pass the workgroups wait for each other: at most 64 of at most
// 80 KB, and bounded waits, after which the finishing kernel colours the graph.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "gc_device.h"
#include "gc_internal.h"

namespace gc {

namespace {

constexpr int kResBlock = 1024;
constexpr int kPack = 6;                            // states to a word
constexpr int kChunkWords = (kWave + kPack - 1) / kPack;
constexpr int kResLanes = 8;                        // lanes per own vertex

// LDS layout: the states of every vertex (whole chunks), the own rows' entries,
// and per own vertex the start of its row.
struct ResLayout {
  int chunks, own_chunks, entries;
  __host__ __device__ ResLayout(int n, int groups, int lds) {
    chunks = (n + kWave - 1) / kWave;
    own_chunks = (chunks + groups - 1) / groups;
    entries = (lds - chunks * kWave - (own_chunks * kWave + own_chunks) * 4) / 2;
  }
};

// Reads the words p[i[k]] (k in want) until each carries `tag`, all of them in
// flight together; false when the wait was given up.
template <int K>
__device__ __forceinline__ bool poll_words(const uint64_t* p, const int* i, uint32_t want,
                                           uint32_t tag, Ctrl* c, int polls, uint64_t* x) {
  long spins = 0;
  while (want) {
#pragma unroll
    for (int k = 0; k < K; ++k)
      if ((want >> k) & 1)
        x[k] = __hip_atomic_load(&p[i[k]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (((want >> k) & 1) && (uint32_t)(x[k] >> 48) == tag) want &= ~(1u << k);
    if (!want) break;
    if (++spins >= polls)
      __hip_atomic_store(&c->abort.v, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((spins & 1023) == 0 &&
        __hip_atomic_load(&c->abort.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      return false;
  }
  return true;
}

__device__ __forceinline__ void publish(uint64_t* p, uint32_t tag, uint64_t x) {
  __hip_atomic_store(p, ((uint64_t)tag << 48) | x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Clears the exchange words, and workgroup g checks that the rows of workgroup
// g of the colouring fit its LDS (core_fail otherwise; the caller looks at it in
// the first call of the pass on a graph).
template <typename RP>
__global__ __launch_bounds__(kWave) void k_res_prepare(KArgs a, ResArgs r, int lds) {
  const ResLayout lay(a.n, gridDim.x, lds);
  const RP* __restrict__ rp = (const RP*)a.rowptr;
  const int P = gridDim.x;
  for (int i = blockIdx.x * kWave + threadIdx.x; i < (2 + kChunkWords) * lay.chunks; i += P * kWave)
    r.words[i] = 0;
  int64_t sum = 0;
  for (int ch = blockIdx.x + threadIdx.x * P; ch < lay.chunks; ch += kWave * P)
    sum += rp[min(a.n, (ch + 1) * kWave)] - rp[ch * kWave];
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) sum += (int64_t)shfl_xor64((uint64_t)sum, off);
  if (threadIdx.x == 0 && sum > lay.entries) a.ctrl->core_fail.v = 1;
}

// `last` > 0: no round after it.
template <typename RP>
__global__ __launch_bounds__(kResBlock) void k_resident(KArgs a, ResArgs r, int lds, int last) {
  extern __shared__ __align__(16) char smem[];
  __shared__ int base[kResMaxChunks + 1];  // entry where each own chunk's rows start
  __shared__ uint32_t own_win[2 * kResMaxChunks];
  __shared__ int sum;
  const ResLayout lay(a.n, gridDim.x, lds);
  int8_t* const st = (int8_t*)smem;
  int32_t* const off = (int32_t*)(smem + lay.chunks * kWave);
  uint16_t* const ent = (uint16_t*)(off + lay.own_chunks * kWave + lay.own_chunks);
  const RP* __restrict__ rp = (const RP*)a.rowptr;
  const int tid = threadIdx.x, lane = lane_id();
  const int g = blockIdx.x, P = gridDim.x;
  if (a.ctrl->core_fail.v) {  // every vertex is left uncoloured
    for (int v = g * kResBlock + tid; v < a.n; v += P * kResBlock) ((int8_t*)a.st)[v] = -1;
    return;
  }
  const int mine = (lay.chunks - g + P - 1) / P;  // own chunks: g, g + P, ...
  // the state words follow the winner words
  uint64_t* const wins = r.words;
  uint64_t* const states = r.words + 2 * lay.chunks;
  for (int v = tid; v < lay.chunks * kWave; v += kResBlock) st[v] = v < a.n ? -1 : 0;
  if (tid == 0) {
    int at = 0;
    for (int i = 0; i < mine; ++i) {
      const int v0 = (g + i * P) * kWave, v1 = min(a.n, v0 + kWave);
      base[i] = at;
      at += (int)(rp[v1] - rp[v0]);
    }
    base[mine] = at;
  }
  __syncthreads();
  // 65 row starts per own chunk (the last is the chunk's end)
  for (int i = tid; i < mine * (kWave + 1); i += kResBlock) {
    const int ch = i / (kWave + 1), j = i % (kWave + 1);
    const int v0 = (g + ch * P) * kWave;
    off[i] = base[ch] + (int)(rp[min(a.n, v0 + j)] - rp[v0]);
  }
  for (int ch = 0; ch < mine; ++ch) {  // a chunk's rows are consecutive
    const RP from = rp[(g + ch * P) * kWave];
    const int len = base[ch + 1] - base[ch];
    for (int i = tid; i < len; i += kResBlock) ent[base[ch] + i] = (uint16_t)a.colidx[from + i];
  }
  int left = a.n;  // uncoloured vertices of the graph
  int own = 0;     // and of this workgroup
  for (int i = 0; i < mine; ++i) own += min(kWave, a.n - (g + i * P) * kWave);
  int rounds = 0;
  const int gl = lane & (kResLanes - 1);
  const uint64_t gmask = ((1ull << kResLanes) - 1) << (lane & ~(kResLanes - 1));
  for (uint32_t q = 1;; ++q) {
    for (int i = tid; i < 2 * mine; i += kResBlock) own_win[i] = 0;
    if (tid == 0) {
      sum = 0;
      const int rd = rounds + 1;
      if (rd <= kTraceRounds) a.ctrl->trace[rd - 1] = left;  // (the same from every workgroup)
    }
    __syncthreads();
    ++rounds;
    // detect: a group of lanes per own vertex (wave-uniform loop)
    for (int i0 = 0; i0 < mine * kWave; i0 += kResBlock / kResLanes) {
      const int i = i0 + tid / kResLanes;
      const int ch = i / kWave, v = i < mine * kWave ? (g + ch * P) * kWave + i % kWave : 0;
      const int s = i < mine * kWave ? (int)st[v] : 0;
      bool hit = false;
      if (s < 0) {
        const int b = off[i + ch], e = off[i + ch + 1];
        for (int k = b + gl; k < e; k += kResLanes) {
          const int u = ent[k];
          hit |= u < v && st[u] == s;  // (uncoloured, the same tentative colour)
        }
      }
      const bool lose = (__ballot(hit) & gmask) != 0;
      if (s < 0 && !lose && gl == 0) {
        atomicOr(&own_win[2 * ch + (v % kWave) / 32], 1u << (v % 32));
        ((int8_t*)a.st)[v] = (int8_t)~s;
      }
    }
    __syncthreads();
    // winners: words with an uncoloured vertex (32 states: none negative?)
    auto open32 = [&](int w) {
      const int4* p = (const int4*)(st + 32 * w);
      const int4 x = p[0], y = p[1];
      return ((x.x | x.y | x.z | x.w | y.x | y.y | y.z | y.w) & 0x80808080) != 0;
    };
    for (int i = tid; i < 2 * mine; i += kResBlock) {
      const int w = 2 * (g + (i / 2) * P) + (i & 1);
      if (open32(w)) publish(&wins[w], q, own_win[i]);
    }
    for (int i = 0; i < 2 * mine; ++i) own -= __popc(own_win[i]);
    if (own == 0) break;  // workgroup-uniform, and before anything is polled
    __syncthreads();  // (all words of st are looked at before any changes)
    int bad = 0, won = 0;
    for (int w0 = tid; w0 < 2 * lay.chunks; w0 += 2 * kResBlock) {
      const int w[2] = {w0, w0 + kResBlock};
      uint64_t x[2] = {0, 0};
      uint32_t want = 0;
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (w[k] < 2 * lay.chunks && open32(w[k])) want |= 1u << k;
      if (!poll_words<2>(wins, w, want, q, a.ctrl, r.polls, x)) bad = 1;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        uint32_t m = (uint32_t)x[k];
        won += __popc(m);
        while (m) {
          const int v = 32 * w[k] + __builtin_ctz(m);
          m &= m - 1;
          st[v] = (int8_t)~st[v];
        }
      }
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) won += __shfl_xor(won, o);
    if (lane == 0 && won) atomicAdd(&sum, won);
    if (__syncthreads_or(bad)) return;
    left -= sum;
    // speculate: own vertices still uncoloured
    for (int i0 = 0; i0 < mine * kWave; i0 += kResBlock / kResLanes) {
      const int i = i0 + tid / kResLanes;
      const int ch = i / kWave, v = i < mine * kWave ? (g + ch * P) * kWave + i % kWave : 0;
      const bool act = i < mine * kWave && st[v] < 0;
      uint64_t lo = 0, hi = 0;
      if (act) {
        const int b = off[i + ch], e = off[i + ch + 1];
        for (int k = b + gl; k < e; k += kResLanes) {
          const int c = st[ent[k]];
          if (c >= 64) hi |= 1ull << (c - 64);
          else if (c >= 0) lo |= 1ull << c;
        }
      }
      if (__ballot(act)) {
        lo = group_or<kResLanes>(lo);
        hi = group_or<kResLanes>(hi);
        // (own uncoloured states are read by their own group alone here)
        if (act && gl == 0)
          st[v] = (int8_t)~(~lo ? __builtin_ctzll(~lo) : 64 + __builtin_ctzll(~hi));
      }
    }
    __syncthreads();
    if (last > 0 && rounds >= last) break;
    // states: words with an uncoloured vertex
    auto open6 = [&](int ch, int j) {
      bool o = false;
#pragma unroll
      for (int k = 0; k < kPack; ++k)
        o |= kPack * j + k < kWave && st[ch * kWave + kPack * j + k] < 0;
      return o;
    };
    for (int i = tid; i < mine * kChunkWords; i += kResBlock) {
      const int ch = g + (i / kChunkWords) * P, j = i % kChunkWords;
      if (!open6(ch, j)) continue;
      uint64_t x = 0;
#pragma unroll
      for (int k = 0; k < kPack; ++k)
        if (kPack * j + k < kWave) x |= (uint64_t)(uint8_t)st[ch * kWave + kPack * j + k] << (8 * k);
      publish(&states[ch * kChunkWords + j], q, x);
    }
    constexpr int kFly = 4;
    for (int i0 = tid; i0 < lay.chunks * kChunkWords; i0 += kFly * kResBlock) {
      int i[kFly];
      uint64_t x[kFly];
      uint32_t want = 0;
#pragma unroll
      for (int f = 0; f < kFly; ++f) {
        i[f] = i0 + f * kResBlock;
        const int ch = i[f] / kChunkWords;
        if (ch < lay.chunks && ch % P != g && open6(ch, i[f] % kChunkWords)) want |= 1u << f;
      }
      if (!poll_words<kFly>(states, i, want, q, a.ctrl, r.polls, x)) bad = 1;
#pragma unroll
      for (int f = 0; f < kFly; ++f) {
        if (!((want >> f) & 1)) continue;
        const int ch = i[f] / kChunkWords, j = i[f] % kChunkWords;
#pragma unroll
        for (int k = 0; k < kPack; ++k)
          if (kPack * j + k < kWave) st[ch * kWave + kPack * j + k] = (int8_t)(x[f] >> (8 * k));
      }
    }
    if (__syncthreads_or(bad)) return;
  }
  if (tid == 0) atomicMax(&a.ctrl->last_round.v, rounds);
  if (own == 0) return;
  // a bounded run: what is left stays uncoloured
  for (int i = tid; i < mine * kWave; i += kResBlock) {
    const int v = (g + (i / kWave) * P) * kWave + i % kWave;
    if (v < a.n && st[v] < 0) ((int8_t*)a.st)[v] = st[v];
  }
}

template <typename RP>
int launch_resident_t(const KArgs& a, const ResArgs& r, int last, int groups, hipStream_t s) {
  const int rc = allow_lds((const void*)&k_resident<RP>, kResLds);
  if (rc) return rc;
  hipLaunchKernelGGL((k_res_prepare<RP>), dim3(groups), dim3(kWave), 0, s, a, r, kResLds);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return (int)e;
  hipLaunchKernelGGL((k_resident<RP>), dim3(groups), dim3(kResBlock), kResLds, s, a, r, kResLds,
                     last);
  return (int)hipGetLastError();
}

}  // namespace

size_t resident_bytes(int64_t n) {
  return (size_t)((n + kWave - 1) / kWave) * (2 + kChunkWords) * sizeof(uint64_t);
}

static int resident_groups(int64_t n) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(kResGroups, (n + kWave - 1) / kWave));
}

bool resident_fits(int64_t n, int64_t m, int sbytes) {
  if (sbytes != 1 || n < 1 || n > kResMaxChunks * (int64_t)kResGroups * kWave) return false;
  const int groups = resident_groups(n);
  const ResLayout lay((int)n, groups, kResLds);
  // a quarter more than the average workgroup's rows: the chunks' sizes differ
  return lay.entries > 0 && m + m / 4 <= (int64_t)lay.entries * groups;
}

int launch_resident(const KArgs& a, bool rp64, const ResArgs& r, int last, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const int groups = resident_groups(a.n);
  return rp64 ? launch_resident_t<int64_t>(a, r, last, groups, s)
              : launch_resident_t<int32_t>(a, r, last, groups, s);
}

}  // namespace gc
