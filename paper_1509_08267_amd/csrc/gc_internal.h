// gc_internal.h -- shared between the C-ABI engine and the gfx950 kernels.
//
// State encoding (one signed integer per vertex, of width S = int8, int16 or
// int32 chosen from the maximum degree):
//   s >= 0   the vertex's colour is final (= s)
//   s <  0   the vertex is still being coloured; its tentative colour of the
//            current round is ~s (so the initial -1 means "tentative 0")
// Every colour and tentative colour is at most deg(v) (First Fit picks the
// least of deg(v) + 1 candidates), so S = int8 holds any graph with maximum
// degree <= 126 and int16 any with maximum degree <= 32766 (the type's least
// value stays spare: it marks a vertex that waits under the id-priority
// schedule).
// A round's speculate phase rewrites only negative entries (negative stays
// negative), and its detect phase turns a winner's ~t into t.  A reader that
// decodes (s < 0 ? ~s : s) therefore sees the same tentative colour before and
// after a concurrent commit, which is what lets detect and commit share one
// pass.
#pragma once
#include <cstdint>

namespace gc {

constexpr int kWave = 64;           // CDNA wavefront width
constexpr int kBlock = 256;         // threads per workgroup of the round kernels
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kTraceRounds = 65536; // rounds whose |U_r| is recorded
constexpr int kHeavyWindow = 4096;  // LDS colour window of the block-per-vertex path (bits)
constexpr int kPushColors = 32;     // colours tracked per vertex by pushed flags
constexpr int kWideColors = 480;    // further colours (32..511) tracked for medium/heavy vertices
constexpr int kSparseChunk = 32;    // detect: at most this many uncoloured vertices in a chunk
                                    // -> a group of lanes each (at least 2)
constexpr int kMaxBlocksPerCu = 64; // workgroups per CU of any round kernel (option limit)
constexpr int kFinishBlocks = 512;  // most workgroups of the finishing pass (one stats pair each)
constexpr int kDeferRow = 512;      // a wavefront- or workgroup-class winner with more row entries
                                    // than this left to push queues them for the grid-wide push pass
constexpr int kPieceEntries = 1024; // row entries of one piece of that pass: one workgroup,
                                    // four entries per thread in flight, one step
constexpr int kFinishHeader = 7;   // its leading output words (see launch_finish)
constexpr int kFinishWords = kFinishHeader + 2 * kFinishBlocks;

// One 128-byte line per field that different blocks write, so that flags and
// counters never share a line.
struct alignas(128) Line {
  int32_t v;
  int32_t pad[31];
};

// Which degree classes still have uncoloured vertices in a round (1 = yes or
// not known to be none): a pass skips a class with none.
struct alignas(128) ClassLine {
  int32_t light, medium, heavy;
  int32_t pad[29];
};

struct Ctrl {
  Line more[3];          // slot r % 3 == 1 when round r has uncoloured vertices
  ClassLine cls[3];      // slot r % 3: the classes with uncoloured vertices in round r
  Line last_round;       // last round that had uncoloured vertices
  Line round_base;       // first round of the next graph of a chunk
  Line bar;              // grid barrier arrivals (monotonic within a launch)
  Line abort;            // set when a wait for other workgroups exceeded its limit
  Line left;             // vertices still uncoloured after the last round
  Line epoch;            // value marking this call's pushed colour flags (1..255)
  Line pend;             // round whose per-workgroup counts in KArgs::part are not yet in
                         // trace (0: none)
  Line pend_grid;        // workgroups of that round's detect pass
  Line core_n;           // vertices of the core pass (gc_core.hip)
  Line core_fail;        // it gave up: a colour beyond its masks
  Line ticket;           // next unit of the data-flow pass (GC_ALGO_SEQ)
  Line over;             // its vertices of a round beyond the trace
  Line tasks;            // 64-bit: push tasks (high half) and their pieces (low half)
                         // queued by this round's detect pass (KArgs::tasks)
  int32_t trace[kTraceRounds];  // |U_r| at slot r - 1
};

// A winner's pushes handed to the grid-wide push pass: colour t to the row
// entries [b, e) (to the list entries lst[b, e) when t carries kFromList),
// cut into pieces first .. first + ceil((e - b) / kPieceEntries) - 1 of the
// pass's piece numbering.
constexpr int32_t kFromList = 1 << 30;

struct PushTask {
  int64_t b;
  int64_t e;
  int32_t t;
  int32_t first;
};

// Arguments of every round kernel.
struct KArgs {
  const void* rowptr;     // int32 or int64, n + 1
  const int32_t* colidx;  // nnz
  void* st;               // n entries of the state type
  int32_t* colors;        // n, the caller's output (the widened state)
  int32_t n;
  int32_t light_max;      // deg <= light_max: a group of L lanes per vertex
  const int32_t* mlist;   // medium vertices (light_max < deg < heavy): a wavefront each
  int32_t mcount;
  const int32_t* hlist;   // heavy vertices: a whole workgroup each
  int32_t hcount;
  int32_t sorted;         // rows ascending: the conflict scan may stop early
  int32_t push;           // forbidden colours pushed by committing neighbours
  int32_t seq;            // id-priority First Fit: speculate picks the vertices whose lower
                          // neighbours are all final, detect commits them (no conflicts)
  uint8_t* seen;          // ceil(n / 64) * 64 * kPushColors: byte c of v == epoch when a
                          // neighbour of v has final colour c (plain byte stores, no atomics);
                          // at flag_index(v, c) (gc_device.h)
  int32_t flags_by_chunk; // flag layout: 1 = colour-major within each 64-vertex chunk (only
                          // when there are no medium or heavy vertices), 0 = 32 bytes per vertex
  int32_t epoch;          // epoch of this call (written to ctrl by the init kernel)
  int32_t clear_seen;     // the init kernel zeroes `seen` and `wide` (first call, epoch wrap)
  int32_t clear_trace;    // the init kernel zeroes ctrl->trace (p-block passes add into it)
  uint8_t* wide;          // (mcount + hcount) * kWideColors flags for colours 32..511
  int32_t wide_clear;     // wide blocks allocated: the init kernel's clear covers all of them,
                          // so a block left over from a larger degree-class split of an
                          // earlier call cannot keep a byte equal to a later epoch
  const int32_t* widx;    // n: index of v's wide flag block, -1 for light vertices
  int32_t* skip;          // n: lower neighbours before this offset of v's row are final
                          // (sorted rows); zeroed by round 1
  int32_t* lst;           // nnz, parallel to colidx: each medium or heavy vertex's list of lower
                          // neighbours not yet seen final (detect_wave_list, detect_block_list),
                          // at its row's offset; null unless the push algorithm runs on sorted
                          // rows with such vertices
  int32_t* llen;          // n: length of that list; zeroed by round 1 with skip
  int32_t* part;          // cus * kMaxBlocksPerCu: active vertices of each workgroup of the
                          // last detect pass; the next pass folds them into ctrl->trace
  PushTask* tasks;        // 2 * (mcount + hcount): pushes of long rows or lists queued by a
                          // detect pass for the grid-wide push pass that follows it (push
                          // algorithm with medium or heavy vertices, not in the persistent
                          // kernel; null otherwise)
  Ctrl* ctrl;
};

// Scratch of the core pass (gc_core.hip).
constexpr int kCoreMax = 4096;  // core vertices at most
constexpr int kCoreColors = 512;  // colours with a mask bit: beyond them the pass gives up
constexpr int kCoreGrid = 256;  // workgroups of the collecting pass at most
struct CoreArgs {
  int32_t* ids;      // kCoreMax: the core vertices in id order
  int32_t* part;     // kCoreGrid: uncoloured vertices per workgroup of the collecting pass
  uint64_t* tents;   // kCoreMax / 2: published tentative colours, round << 32 | two of them
  uint64_t* wins;    // 2 * kCoreMax / 64: published winners, round << 32 | 32 of them
  int32_t polls;     // polls after which a wait gives up
};
constexpr size_t kCoreBytes = (size_t)kCoreMax * 4 + kCoreGrid * 4 + (size_t)kCoreMax / 2 * 8 +
                              (size_t)2 * (kCoreMax / 64) * 8;
// The uncoloured vertices of a.st become the core (ctrl->core_n of them).
int launch_core_collect(const KArgs& a, int sbytes, const CoreArgs& c, void* stream);
// The remaining rounds, the first of them round0 + 1 and none after round
// `last` (0: no bound), by 64 core vertices per workgroup; ctrl->core_fail says
// when it gave up (vertices stay uncoloured).
int launch_core(const KArgs& a, bool rp64, int sbytes, const CoreArgs& c, int round0, int last,
                int workgroups, void* stream);
// The resident pass (gc_resident.hip).
constexpr int kResGroups = 64;         // workgroups at most
constexpr int kResMaxChunks = 6;       // 64-vertex chunks of one at most: 24,576 vertices
constexpr int kResLds = 78 * 1024;     // LDS of one (two to a compute unit)
struct ResArgs {
  uint64_t* words;  // resident_bytes(n): the published words
  int32_t polls;    // polls after which a wait gives up
};
size_t resident_bytes(int64_t n);
// Whether a graph's rows (on average) and states fit; one-byte states only.
bool resident_fits(int64_t n, int64_t m, int sbytes);
// The whole colouring, states into a.st (all of them written unless `last` > 0
// stops it), rounds and round sizes into ctrl; ctrl->core_fail is set and
// nothing else done when a workgroup's rows don't fit.
int launch_resident(const KArgs& a, bool rp64, const ResArgs& r, int last, void* stream);

// 32-bit row pointers as 64-bit ones.
int launch_widen_rowptr(const int32_t* rowptr, int64_t n, int64_t* out, void* stream);

// Every vertex uncoloured with tentative colour 0 (what precedes round 1).
int launch_fill_tent0(const KArgs& a, int sbytes, int grid, void* stream);

// Arguments of the data-flow pass of the id-priority schedule (gc_seq.hip).
struct FlowArgs {
  const void* rowptr;     // int32 or int64, n + 1
  const int32_t* colidx;  // nnz
  void* word;             // n words, uint32 or (wide) uint64: 0, or (round << cbits) | colour
  int32_t* colors;        // n, the caller's output
  int32_t n;
  int32_t light_max;      // deg <= light_max: a lane per vertex, above: a wavefront
  int32_t sorted;         // rows ascending: a row is read up to its first id above the vertex
  int32_t wide;           // 64-bit words (cbits = 32): colours and rounds don't fit 32 bits together
  int32_t last;           // > 0: vertices of a later round are reported uncoloured
  int32_t cbits;          // bits of a colour (at most the maximum degree) in a word
  const int32_t* starts;  // first id of each unit, and n behind the last
  const int32_t* units;   // their number
  Ctrl* ctrl;
};
constexpr int kUnitGrid = 256;  // workgroups of the passes that build the units

// The units for `a`'s graph and light_max: their first ids into `starts`
// (room for one per 64 vertices and two per vertex of degree above light_max,
// and one), their number into `units`; `part` holds kUnitGrid words.
int launch_flow_units(const FlowArgs& a, bool rp64, int32_t* part, int32_t* starts, int32_t* units,
                      int grid, void* stream);
int launch_flow_clear(const FlowArgs& a, int grid, void* stream);
int launch_flow(const FlowArgs& a, bool rp64, int grid, void* stream);
// Writes the caller's colours, the trace and `out` (as launch_finish).
int launch_flow_finish(const FlowArgs& a, int32_t* out, void* stream);

// Arguments of the p-block kernels (GC_ALGO_BLOCKS, gc_blocks.hip).
struct BArgs {
  const void* rowptr;     // int32 or int64, n + 1
  const int32_t* colidx;  // nnz
  int32_t* color;         // n: current colours (-1 before a vertex's first), the caller's output
  int32_t* slot;          // nnz: ForbiddenColors slot of each entry whose neighbour is in
                          // another block (entries within a block are not used)
  uint8_t* todo;          // n: 1 while the vertex is to be (re)coloured
  int32_t n;
  int64_t p;              // blocks
  int32_t round;          // round being run (1-based), for the trace
  Ctrl* ctrl;
  // the passes that keep masks in the place of the slots (maximum degree at
  // most 126, at most kBlkMaxVertices vertices per block)
  int8_t* st;             // n: current colours, -1 before a vertex's first
  uint64_t* mask;         // 2n: colours of the neighbours in other blocks after the last round
                          // (bit c of the 128), of the vertices still to be (re)coloured
  uint64_t* nb;           // words * n: neighbours in the vertex's own block, bit j the j-th
                          // vertex of its unit
  int32_t words;          // 64-vertex words of a unit
  int64_t unit;           // blocks of a unit
  int32_t* part;          // active vertices of each workgroup of the last phase 2
  int32_t count_left;     // phase 2 adds the vertices to recolour into ctrl->left
};
constexpr int kBlkMaxVertices = 256;

int launch_blocks_init(const BArgs& a, bool rp64, int grid, void* stream);
// Phase 1 (phase = 1) or phase 2 (phase = 2) of one round; after phase 2,
// ctrl->left holds the vertices to recolour and ctrl->trace / last_round the
// round's size.
int launch_blocks_phase(const BArgs& a, bool rp64, int phase, int grid, void* stream);
// The same passes with masks: the in-block neighbours (once per call, before
// round 1), then phase 1 or phase 2 of round a.round.  A phase of a round with no
// vertex to recolour (ctrl->more) does nothing.
int launch_blkm_init(const BArgs& a, bool rp64, int grid, void* stream);
int launch_blkm_phase(const BArgs& a, bool rp64, int phase, int grid, void* stream);
// ctrl->left = value (vertices still to recolour when a round cap stops the loop)
int launch_blocks_set_left(Ctrl* c, int value, void* stream);

// Relabelling by a vertex order (gc_order.hip).  Writes the relabelled CSR
// (rows ascending) into rowptr2 (n + 1 entries of the input's width) and
// colidx2 (nnz), and newid[v] = the new id of v.  Synchronises `stream`.
int build_order(const void* rowptr, bool rp64, const int32_t* colidx, int32_t n, int64_t nnz,
                int kind, uint64_t seed, void* rowptr2, int32_t* colidx2, int32_t* newid, int grid,
                void* stream);
// out[v] = coloured[newid[v]]
int launch_permute_back(const int32_t* newid, const int32_t* coloured, int32_t n, int32_t* out,
                        int grid, void* stream);

// Records `msg` as the calling thread's last error (gc_last_error(NULL)).
void set_thread_error(const char* msg);

// Launch helpers implemented in gc_kernels.hip.  All return a hipError_t
// cast to int.  `sbytes` is the state width in bytes (1, 2 or 4).
int launch_init(const KArgs& a, void* stream);
int launch_round1(const KArgs& a, bool rp64, int sbytes, int lanes, int grid, void* stream);
// A graph of kernels in the making, each behind the one before (hipGraph_t, hipGraphNode_t).
struct KernelChain {
  void* graph;
  void* last;  // null before the first
};
// With a chain the kernels become nodes of its graph and the stream is not used.
int launch_round(const KArgs& a, bool rp64, int sbytes, int lanes, int phase /*0 spec, 1 detect*/,
                 int round, bool round_from_base, int grid, void* stream,
                 KernelChain* chain = nullptr);
int launch_advance_base(const KArgs& a, int by, void* stream, KernelChain* chain = nullptr);
// Into pinned memory, after round `round`: out[0] whether vertices are left,
// out[1] the round's size |U_round|.
int launch_report(const KArgs& a, int round, int32_t* out, void* stream);
// The state becomes the caller's int32 colours.  `out` (kFinishWords words of
// device-visible pinned host memory) receives, by system-scope stores:
//   out[0] last round, out[1] abort flag, out[2] uncoloured count recorded by
//   earlier passes (ctrl->left), out[3] workgroups G of this pass, out[4]
//   whether the core or resident pass could not run, out[5] the round after which
//   a core pass could take over (the first one that leaves at most kCoreMax
//   vertices; -1 if there is none, or without `find_core`), out[6] the vertices
//   it leaves, and for each workgroup b < G: out[7 + 2b] = its largest colour + 1
//   (0 if none), out[8 + 2b] = its uncoloured vertices.
// The host folds them once the stream has passed this kernel.
int launch_finish(const KArgs& a, int sbytes, bool find_core, int32_t* out, void* stream);

// After a core or resident pass whose result nobody looks at before it is used:
// when a wait in it gave up (ctrl->abort), the vertices it had are coloured again
// by this kernel's first workgroup alone, which waits for nobody, and out[4] is
// kRecoloured, out[1] 0.
constexpr int kRecoloured = 2;
struct AloneArgs {
  const int32_t* ids;  // the ctrl->core_n vertices of a core pass in id order, or null: all
  int32_t round0;      // the rounds start after it
  int32_t last;        // and none follows `last` (0: no bound)
  int32_t rp64;
};
int launch_finish_fused(const KArgs& a, int sbytes, const AloneArgs& w, int32_t* out, void* stream);
int launch_persistent(const KArgs& a, bool rp64, int sbytes, int lanes, int max_rounds, int grid,
                      void* stream);
int persistent_max_grid(bool rp64, int sbytes, int lanes, int* grid_out);
int launch_classify(const void* rowptr, bool rp64, int32_t n, int32_t light_max, int32_t heavy_min,
                    int32_t* mlist, int32_t* hlist, int32_t* counts /*[3]: medium, heavy, maxdeg*/,
                    int32_t* widx, int grid, void* stream);
int launch_wide_index(const int32_t* hlist, int32_t hcount, int32_t mcount, int32_t* widx,
                      void* stream);
int launch_validate(const void* rowptr, bool rp64, const int32_t* colidx, int32_t n, int64_t m,
                    bool sorted, int32_t* err /*[2]: code, where*/, int grid, void* stream);

}  // namespace gc
