// tpmc_launch.h -- host-side launchers of the HIP kernels (defined in the .hip files).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "tpmc_internal.h"
#include "tpmc_units.hpp"

namespace tpmc {

// Static LDS of batch_kernel beside its traversal stack, at most (queue, rings,
// claims): stacks of up to 32 slots, which have the survivor rings, and larger
// ones.  A host test holds the compiled kernels to it; 32 slots with their tallies
// fit four times into a compute unit's 160 KB by 160 bytes each.
constexpr uint32_t kBatchLdsPrecull = 7808, kBatchLds = 6784;

}  // namespace tpmc

namespace tpmc {

// Tally strategy of the trace kernels.
// Auto: per query, global per-triangle atomics or register totals (serving steps
// that mix both kinds of request).
enum TallyMode { kTallyGlobal = 0, kTallyLds = 1, kTallyLane = 2, kTallyTotals = 3, kTallyAuto = 4 };

// Copies of the queries' scalar blocks: copy c of query i at
// base + ((i << log2) + c) * kScalStride (base null: none, the block itself is
// added into).  Workgroup b adds into copy b % 2^log2, finalize_kernel sums
// them.  One address takes an atomic every 12 ns, so the 12 sums of each of
// 4096 waves on one block took 355 us; workgroups b, b + 8, ... run on one XCD,
// so a copy's cache line also stays in that XCD's L2 (eight copies: 49 us).
struct ScalCopies {
  long long* base;
  uint32_t log2;
};

// Copies of the per-triangle tallies: copy c of the words [0, stride) at
// base + c * stride (base null: none).  Workgroup b adds into copy b % 2^log2;
// the reduction sums them.
struct TallyCopies {
  long long* base;
  uint32_t log2;
  uint64_t stride;
};

// A launch covers the queries qs[0, gridDim.y) of one tally kind (the others'
// workgroups leave at once), workgroups x of query y.
struct TraceArgs {
  const Node* nodes;
  const TriRec* tris;
  const uint32_t* orig;
  const QueryDev* qs;         // device pointer
  const float* x[3];          // SoA planes
  const float* w[3];
  long long* tally;           // indexed by QueryDev::tally_offset
  long long* scal;            // indexed by QueryDev::scalar_offset
  ScalCopies copies;          // of the blocks of qs
  TallyCopies tally_copies;   // of the words at tally
  int32_t* first_tri;         // optional, indexed by QueryDev::p_offset
  unsigned long long* counters;  // optional [2]: BVH nodes visited, triangle tests
  uint32_t nt;
  uint32_t refill;            // serve ended segments when fewer lanes of a wave traverse (1..64)
};

// One persistent launch covers n_entries entries; entry j is entry_tiles[j]
// tiles of query entry_query[j] starting at tile entry_tile0[j] (a serving
// step: any slots, any ranges), or, with null lists, all particles of query j
// (a whole batch).  Each entry is cut into 2^sub_log2 parts with a claim
// counter each (entry_next[j << sub_log2 | part]), so that the waves of a
// launch with few queries do not all claim from one address (12 ns per atomic
// on one address, measured).  A part is handed out in units of whole
// 64-particle batches (UnitPlan in tpmc_units.hpp): one unit per wave that
// starts on it (StartPlan there), taken without an atomic, then units by the counter
// that halve in size towards the part's end.  A wave stays on one query and flushes its
// partial sums only when it moves to another.  With workgroup LDS tallies the
// workgroup's waves move to another part together.
struct BatchArgs {
  const QueryDev* qs;              // query / slot table (meshes referenced per query)
  const uint32_t* entry_query;     // [n_entries] or null (entry j is query j)
  const uint64_t* entry_tile0;     // [n_entries] or null (start at tile 0)
  const uint64_t* entry_tiles;     // [n_entries] or null (every tile of the query)
  unsigned long long* entry_next;  // [n_entries << sub_log2] claim counters, zeroed before the launch
  long long* tally_base;           // per-triangle tallies, indexed by QueryDev::tally_offset
  long long* scal_base;            // scalar blocks, indexed by QueryDev::scalar_offset
  ScalCopies copies;               // of the blocks of qs
  TallyCopies tally_copies;        // of the words at tally_base
  uint32_t n_entries;
  uint32_t sub_log2;               // parts per entry (log2)
  uint32_t refill;                 // as TraceArgs::refill
  uint32_t tile;                   // particles per tile (multiple of 64)
  uint32_t unit_cap_log2;          // no unit exceeds 64 << unit_cap_log2 particles (<= 8: 16-bit offsets in a unit)
  uint32_t share_log2;             // particles per wave of the whole launch (log2, rounded down)
  StartPlan start;                 // the parts that workgroups start on without an atomic (own 0, div 0: none)
  uint32_t start_cap_log2;         // no starting unit exceeds 64 << start_cap_log2 particles
  uint32_t xcd_cus;                // compute units per XCD
  uint32_t lds_tris;               // largest nt of an entry with an LDS tally (kTallyLds / kTallyAuto)
  uint32_t wave_totals;            // kTallyAuto: some entry keeps totals only (per-wave LDS totals allocated)
  // Where each XCD's workgroups start claiming without a starting part: XCD x
  // (workgroups x, x + 8, ...; the hardware deals workgroups to the eight XCDs
  // in turn) starts in entries [xcd_start[x], xcd_start[x + 1]) (entries
  // grouped by mesh, ranges by tile share), so that each XCD's L2 holds the
  // hierarchies of few meshes.
  uint32_t xcd_start[9];
};

// Word ranges cleared by one launch (n 0: none).
constexpr int kClearRanges = 5;
struct ClearRanges {
  long long* p[kClearRanges];
  uint64_t n[kClearRanges];
};
void clear_ranges(const ClearRanges& r, hipStream_t st);
// The same, and writes the n <= kArgQueries queries at h_qs (copied into the
// launch's arguments) to d_qs: no copy, no host memory to keep, no wait.
constexpr uint32_t kArgQueries = 4;
void clear_and_upload(const ClearRanges& r, const QueryDev* h_qs, QueryDev* d_qs, uint32_t n, hipStream_t st);
void zero_i64(long long* p, uint64_t n, hipStream_t st);
// Fills the seeding start table of the current device (once per device).
hipError_t init_seed_tables(hipStream_t st);
void zero_u32(uint32_t* p, uint64_t n, hipStream_t st);

// What the host reads of a build.
struct BuildRead {
  Node root;
  uint32_t depth;  // 0: the builder gave it
};
// Supporting-plane flags in bits 30 / 31 of orig[] (after a build; see
// tpmc_bvh.hip), and the build's result at d_read (depth from d_depth unless null).
size_t support_scratch_bytes(uint64_t nt);
void mark_support(const float* d_xyz, uint64_t nv, const TriRec* d_tris, uint64_t nt, uint32_t* d_orig,
                  const Node* d_nodes, const uint32_t* d_depth, BuildRead* d_read, void* scratch, hipStream_t st);
constexpr uint32_t kOrigIdMask = 0x3FFFFFFFu;  // orig[] bits 0..29: original triangle index
// Enqueued only; the depth is at *d_depth once the stream has run (null: *h_depth has it).
size_t bvh_scratch_bytes(uint64_t nt);
hipError_t build_bvh(const float* d_xyz, const uint32_t* d_tri, uint64_t nt, const float box_lo[3],
                     const float box_hi[3], void* scratch, Node* d_nodes, TriRec* d_tris, uint32_t* d_orig,
                     uint32_t* h_depth, const uint32_t** d_depth, hipStream_t st);

// Top-down binned-SAH hierarchy in the same node / leaf format (default builder).
size_t sah_scratch_bytes(uint64_t nt);
hipError_t build_bvh_sah(const float* d_xyz, const uint32_t* d_tri, uint64_t nt, void* scratch, Node* d_nodes,
                         TriRec* d_tris, uint32_t* d_orig, uint32_t* h_depth, hipStream_t st);

int stack_slots_for_depth(uint32_t depth);  // 0 when too deep
// Plain path: one launch of up to kMaxGridY queries each, max_n particles in the largest.
constexpr uint32_t kMaxGridY = 65535;
void launch_seed(const QueryDev* d_qs, uint32_t nq, uint64_t max_n, float* const planes[6], int n_cu, hipStream_t st);
void launch_trace(const TraceArgs& a, uint32_t nq, uint64_t max_n, int stack_slots, TallyMode mode, int max_grid,
                  hipStream_t st);
// Clears the queries' totals, then sums their triangles (plain path).
void launch_reduce_totals(const QueryDev* d_qs, uint32_t nq, long long* tally_base, long long* scal_base,
                          uint32_t max_nt, hipStream_t st);
// tally_base (null: none): per-triangle tallies that finalize sums itself, of
// meshes of at most kFinalizeTris triangles (their queries' totals in scal are zero).
constexpr uint32_t kFinalizeTris = 2048;
constexpr uint32_t kMaxFinalize = 65536;  // queries of one launch, a workgroup each
void launch_finalize(const QueryDev* d_qs, const uint32_t* d_idx, const long long* scal_base, const ScalCopies& copies,
                     const long long* tally_base, const TallyCopies& tally_copies, uint32_t nq, double xr, double yr,
                     double zr, double A_ref, ResultDev* out, hipStream_t st);
void launch_reduce_slots(const QueryDev* d_qs, const uint32_t* d_idx, uint32_t n, long long* tally_base,
                         long long* scal_base, uint32_t max_nt, hipStream_t st);
// Launches at most groups_per_cu workgroups per compute unit over total_particles: no
// more than are resident at once and no more than there are batches (or, in a batch,
// queries) for.  uniform: every entry may be started on without an atomic (a
// batch); sub_log2, the shares and the starting parts of a are set here; counters:
// words at a.entry_next.
void launch_batch(BatchArgs a, int stack_slots, TallyMode mode, uint64_t total_particles, bool uniform,
                  uint64_t counters, int n_cu, int groups_per_cu, hipStream_t st);
// Check of the two-stage seeding's estimate (precull_check_kernel): out[0] the
// bits of the largest error / margin, out[1] the particles estimated.
void launch_precull_check(const QueryDev* d_q, uint64_t n, unsigned long long* out, int grid, hipStream_t st);
// Phase probe: whether this library was built with it; the readout copies the
// kProbeSlots sums of the current device into out (after the stream's work)
// and clears them when reset.
bool probe_built();
hipError_t probe_read(unsigned long long* out, bool reset, hipStream_t st);
// Fills the own latitude rows (kLatOwnStride floats each) of the queries that have one.
void launch_lat_own(const QueryDev* d_qs, uint32_t nq, float* rows, hipStream_t st);
// Serving admission: n records (device) -> constants into qs[slot], cleared
// scalar block (and copies), per-triangle tally words, and its own latitude row; max_words is the largest tally.
void launch_admit(const AdmitRec* rec, uint32_t n, uint64_t max_words, QueryDev* qs, long long* scal,
                  const ScalCopies& copies, float* lat_rows, long long* tally, hipStream_t st);

// Ceiling microkernels (tpmc_ceilings.hip).  kind 0: FP32 FMA, 1: FP64 FMA,
// 2: int32 multiply and add; each lane performs ceiling_valu_ops_per_lane(iters)
// of them.
void launch_ceiling_valu(uint32_t kind, int grid, uint32_t iters, void* sink, hipStream_t st);
uint64_t ceiling_valu_ops_per_lane(uint32_t iters);
void launch_ceiling_read(const void* p, uint64_t bytes, uint32_t passes, int grid, hipStream_t st);
void launch_ceiling_atomic(void* p, uint32_t slots, uint32_t per_thread, int grid, hipStream_t st);
void launch_ceiling_lds_atomic(void* sink, uint32_t slots, uint32_t per_thread, int grid, hipStream_t st);
void launch_reduce_batch(const QueryDev* d_qs, uint32_t nq, long long* tally_base, const TallyCopies& copies,
                         long long* scal_base, uint32_t max_nt, hipStream_t st);
// tally[0, stride) += the copies, which are cleared.
void launch_fold_tally(long long* tally, const TallyCopies& copies, hipStream_t st);

}  // namespace tpmc
