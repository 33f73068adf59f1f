// Internal host-side interfaces between the translation units of libsfc.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "learned.h"
#include "stree.h"

namespace sfc {

inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Occupancy bitmap of the quadtree nodes of depths 0..kOccDepth (early
// termination): depth k starts at bit (4^k - 1) / 3, node p of depth k (the
// top 2k key bits) at that offset + p.
constexpr int kOccDepth = 12;
__host__ __device__ constexpr uint64_t occ_level_offset(int k) {
  return ((1ull << (2 * k)) - 1) / 3;
}
constexpr uint64_t kOccBits = occ_level_offset(kOccDepth + 1);
constexpr uint64_t kOccWords = (kOccBits + 31) / 32;

// Launch shapes chosen by the autotuner, per size bucket (floor(log2 size)).
// tuned(op, size) returns -1 when the bucket has no entry.
enum TuneOp { kTuneSortItems = 0, kTuneTestShape = 1 };
int tuned(TuneOp op, uint64_t size);
void set_tuned(TuneOp op, uint64_t size, int value);

// Fill kernel (used instead of hipMemsetAsync so that every step of a batch
// can be recorded into a HIP graph).
hipError_t fill_u64(uint64_t* p, uint64_t value, uint64_t count, hipStream_t s);
hipError_t fill_u32(uint32_t* p, uint32_t value, uint64_t count, hipStream_t s);

// ---- construction (build.hip) ----
size_t build_scratch_bytes(uint64_t n);
// Run condition of a kernel sequence recorded beside an alternative one (a
// recorded graph cannot branch on the host): with word != null each of its
// kernels returns at once unless the kErrOversized bit of *word is set
// (when_set) or clear (!when_set).
struct SortGuard {
  const uint32_t* word = nullptr;
  bool when_set = true;
};
// Keys of n points (err: device word, kErrDomain is or-ed in); counts, if
// not null, receives the first digit's counts per sort tile.
hipError_t launch_keys(const double* xy, uint64_t n, int curve, uint64_t* keys, uint32_t* err,
                       uint32_t* counts, hipStream_t s, double* xy_copy = nullptr,
                       int count_shift = 0, SortGuard guard = SortGuard{});
// xy_out (may be null): the points in sorted order.  cells_out (may be
// null): the grid cells of the sorted points (pack_cell2 / pack_cell3),
// decoded from the keys (or taken from the points when they are gathered).
// xy_copy (may be null): a copy of the input points in input order.
hipError_t sort_build(const double* xy, uint64_t n, int curve, uint64_t* keys_out,
                      uint32_t* ids_out, double* xy_out, void* scratch, uint32_t* err,
                      hipStream_t s, const uint64_t* set_off = nullptr, uint32_t n_sets = 0,
                      uint64_t* cells_out = nullptr, double* xy_copy = nullptr,
                      SortGuard guard = {});
// sort_build without point sets, of up to kSmallSort points, in two launches.
constexpr uint64_t kSmallSort = 1u << 16;
hipError_t sort_build_small(const double* xy, uint64_t n, int curve, uint64_t* keys_out,
                            uint32_t* ids_out, double* xy_out, void* scratch, uint32_t* err,
                            hipStream_t s, uint64_t* cells_out, double* xy_copy);
// sort_build without point sets or xy_out, by four radix passes over the
// top 32 key bits and an LDS sort of each chunk of whole runs of equal top
// bits (same results).  A run too long for a chunk raises kErrOversized in
// *err, and the arrays are then unspecified: run sort_build instead.  Same
// scratch as sort_build.
hipError_t sort_build_chunked(const double* xy, uint64_t n, int curve, uint64_t* keys_out,
                              uint32_t* ids_out, void* scratch, uint32_t* err, hipStream_t s,
                              uint64_t* cells_out, double* xy_copy);
// sort_build_chunked with point sets (set_off and n_sets as in sort_build;
// none: the chunked sort alone): the chunked sort of all points by key, then
// stable passes over the set index (so that the order is by set, key, id, as
// sort_build's).  A run too
// long for a chunk raises kErrOversized and the set passes do nothing; with
// fallback the plain sort_build (with the sets) then runs on the device,
// its kernels recorded after these and doing nothing unless the bit is set.
// xy_out (may be null): the points in sorted order.  No host
// synchronisation: the whole sequence can be recorded into a graph.  Same
// scratch as sort_build.
hipError_t sort_build_sets_chunked(const double* xy, uint64_t n, int curve, uint64_t* keys_out,
                                   uint32_t* ids_out, double* xy_out, void* scratch, uint32_t* err,
                                   hipStream_t s, const uint64_t* set_off, uint32_t n_sets,
                                   uint64_t* cells_out, double* xy_copy, bool fallback);
// out[i] = xy[ids[i]] for points of dim (2 or 3) doubles.
hipError_t gather_sorted(const uint32_t* ids, const double* xy, double* out, uint64_t n, int dim,
                         hipStream_t s);
// Order of a batch of m queries (centres clamped into the domain) along the
// curve, as far as the places of their keys among the n >= 1 sorted ones, taken
// to 11 bits, tell: perm[i] = the i-th query in that order.  scratch holds
// order_scratch_bytes(m).  wanted (device, may be null): if it holds 0 when the
// kernels run, they do nothing.
size_t order_scratch_bytes(uint64_t m);
hipError_t order_queries(const double* q, uint64_t m, int curve, const uint64_t* keys, uint64_t n,
                         uint32_t* perm, void* scratch, hipStream_t s,
                         const uint32_t* wanted = nullptr);
// Early-termination occupancy bitmap (kOccWords words) of n sorted keys.
hipError_t build_occupancy(const uint64_t* keys, uint64_t n, uint32_t* occ, hipStream_t s);

// ---- device-wide scan (scan.hip) ----
// out[i] = carry + sum(in[0..i)), out[count] = carry + sum(in); carry_in is a
// device word or null (zero).  partial holds scan_scratch_bytes(count).
size_t scan_scratch_bytes(uint64_t count);
hipError_t scan_excl(const uint32_t* in, uint64_t* out, uint64_t count, const uint64_t* carry_in,
                     uint64_t* partial, hipStream_t s);

// ---- queries (query.hip) ----
// The counters of a batch, in device memory; the compaction's last kernel
// copies them to host memory when asked to.
struct BatchStatus {
  uint64_t rows;         // candidate rows of 64
  uint64_t total;        // reported ids (host copy only)
  uint64_t candidates;
  uint64_t endpoints;    // learned lower bounds
  uint64_t fallbacks;    // of which fell back to binary search
  uint64_t pruned;       // cells skipped by early termination
  uint32_t err;          // kErr* bits
  uint32_t coarse;       // some radius lies past the cell filter's shift limit
  uint32_t units;        // compaction units of the current chunk
  uint32_t left;         // the compaction leaves the batch alone (expand_rows decides)
};

// What the search leaves of each query for the test pass: nothing, the cell
// filter's limits, or the query itself (tests that read every point); for
// queries at epochs also their epoch (qepoch[j], valid in [oldest, epoch], or
// `epoch` when qepoch is null).
enum { kRecordNone = 0, kRecordFilter = 1, kRecordExact = 2 };
struct RecordPlan {
  void* rec = nullptr;
  int mode = kRecordNone;
  bool window = false;
  const uint32_t* qepoch = nullptr;
  uint32_t oldest = 0, epoch = 0;
};

// Scratch of one batch of m queries.  Places are positions in the order that
// the rows are processed in: the queries' own, or the curve order of perm.
struct QueryScratch {
  uint64_t m = 0;
  BatchStatus* status;
  uint2* slots;            // per query and slot: first sorted index, candidates
  uint64_t* row_off;       // per place: its first row (+ the total at [m])
  uint64_t* blk_rows;      // per workgroup of queries: its rows,
  uint64_t* blk_off;       //   its first row,
  uint64_t* blk_stat;      // per search workgroup: its candidates and flags,
  uint64_t* blk_rows64;    //   its rows of 64 candidates,
  uint64_t* blk_place;     //   (queries in curve order) its rows,
  uint32_t* blk_learned;   //   its learned endpoints and fallbacks
  void* groups;            // per group of workgroups: its rows and counters
  void* rec;               // per query: the test pass's record (32 B)
  uint32_t* perm;          // the queries in curve order
  uint64_t* out_base;      // per query: added to the hits before a row gives its output
  uint32_t* qhits;         // per query: its reports
  uint64_t* scan_tmp;      // scan partials
  void* order_scratch;     // order_scratch_bytes(m)
  uint64_t* pairs;         // early termination: dense (query, cell) list, 4 * query + cell
  uint64_t* regions;       //   the same, by workgroup
  uint32_t* pack_cnt;      //   per workgroup: its pairs,
  uint32_t* pack_pre;      //   those before it (+ the total),
  uint32_t* pack_wanted;   //   whether the queries are listed in curve order,
  uint32_t* pack_pruned;   //   its pruned cells,
  uint64_t* pack_flags;    //   its flags
  int ss;                  // log2 of the slots per query
  int block_queries;       // queries per search workgroup
  uint32_t stats_ns, stats_np;   // workgroups whose counters are summed
  bool learned;            // blk_learned is filled
  bool perm_made;          // perm holds the queries in curve order
  bool fused;              // expand_rows scans blk_rows and sums the counters itself
};
constexpr uint64_t kCompactTileRows = 64;           // rows of 64 candidates per tile
constexpr uint64_t kCompactChunkTiles = 1ull << 19; // tiles per launch
// Tiles per chunk in effect (kCompactChunkTiles unless a test lowered it).
uint64_t compact_chunk_tiles();
void set_compact_chunk_tiles(uint64_t tiles);
// Query scratch for m queries of up to `slots` slots each (8: the plane,
// either layout, and three dimensions unrefined; 32: three dimensions
// refined).  The carving returns false if the layout needs more than that.
size_t query_scratch_bytes(uint64_t m, uint32_t slots = 8);
bool query_scratch_carve(void* base, uint64_t m, QueryScratch* qs, uint32_t slots = 8);
size_t compact_scratch_bytes(uint64_t total_rows);

// Ranges and searches of a batch (qs carved for its m queries), then the
// rows and the batch's counters.
struct RangePlan {
  const double* q = nullptr;
  const double* delta = nullptr;
  int dim = 2;                         // 3: points and queries of three doubles, Morton keys
  const uint64_t* keys = nullptr;
  uint64_t n = 0;
  int curve = 0;
  bool refine = false;
  uint32_t refine_min = 0;
  bool ball = false;                   // Euclidean metric: the refinement may drop sub-cells
                                       // outside the disc
  const LearnedView* lview = nullptr;  // search through the learned index; else
  const StreeView* sview = nullptr;    // through the static search tree (not with point sets)
  const uint32_t* occ = nullptr;       // skip cells whose occupancy bit is clear
  const uint32_t* qset = nullptr;      // query j searches only set qset[j] (positions
  const uint64_t* set_off = nullptr;   // [set_off[s], set_off[s+1]) of the sorted arrays)
  uint32_t n_sets = 0;
  double last_candidates = -1.0;       // a query of the handle's last batch (negative: none)
  RecordPlan record;
  bool need_rows = false;              // the caller reads the counters before the compaction
  BatchStatus* host = nullptr;         // receives them then (host memory), if not null
  // Inspection (all or none): the method's key and index ranges, four per
  // query, and their number; no early termination, refinement or records.
  uint64_t* dbg_lo = nullptr;
  uint64_t* dbg_hi = nullptr;
  uint64_t* dbg_b = nullptr;
  uint64_t* dbg_e = nullptr;
  uint32_t* dbg_nr = nullptr;
};
hipError_t launch_ranges(const RangePlan& P, QueryScratch& qs, hipStream_t s);

// Test-and-compact over the candidate rows of a batch whose ranges are in qs.
struct CompactPlan {
  const double* q = nullptr;
  const double* delta = nullptr;
  const double* pts = nullptr;       // the sorted points, or null: then
  const double* pts_in = nullptr;    // the points in input order, read through their ids
  const uint64_t* cells = nullptr;   // grid cells of the sorted points: with them most
                                     // candidates are decided from their cell and only the
                                     // others read their point; without, pts must be set
  const uint32_t* ids = nullptr;
  const uint64_t* keys = nullptr;    // the sorted keys, their number and the curve, to process
  uint64_t n = 0;                    // the rows in curve order; null: in query order
  int curve = 0;
  uint64_t max_rows = 0;             // device_sized false: the exact row count, processed in
  bool device_sized = false;         // chunks; true: a capacity, the count is read on the
                                     // device and more rows raise kErrOverflow
  uint64_t shape_rows = 0;           // the test pass's launch shape is that for so many rows
                                     // (0: for max_rows)
  void* scratch = nullptr;           // compact_scratch_bytes(max_rows)
  uint64_t* offsets = nullptr;
  uint32_t* out_ids = nullptr;
  uint64_t cap = 0;
  bool window = false;               // the square-window test instead of the ball
  int dim = 2;
  const uint32_t* ins = nullptr;     // with both: only entries with ins <= e < era are
  const uint32_t* era = nullptr;     // visible to a query at epoch e
  bool write_only = false;           // the write pass alone, on a batch still in scratch
  uint32_t reject = 0;               // kErr* bits: a batch with one of them is left alone, its
                                     // offsets and ids as they were
  int coarse = -1;                   // BatchStatus::coarse if the caller read it (1, 0), else
                                     // -1; with 0 the test pass takes its shortest form
  BatchStatus* host = nullptr;       // host memory: the final counters, if not null
  uint32_t* flags_out = nullptr;     // device: the final error bits, if not null
};
hipError_t launch_compact(const CompactPlan& P, const QueryScratch& qs, hipStream_t s);
// Whether a batch of total_rows rows is compacted in one chunk: then an output
// larger than the capacity leaves the ids untouched, and the write pass can be
// rerun alone (write_only) for a larger buffer.
bool compact_single_chunk(uint64_t total_rows);
// Scan with the element count in device memory (count_dev <= max_count).
size_t scan_dev_scratch_bytes(uint64_t max_count);
hipError_t scan_excl_dev(const uint32_t* in, uint64_t* out, const uint32_t* count_dev,
                         uint64_t max_count, const uint64_t* carry_in, uint64_t* partial,
                         hipStream_t s);

// ---- updates (update.hip) ----
constexpr uint32_t kLiveEpoch = 0xFFFFFFFFu;   // era of an entry not erased
// The stored run: sorted (key, id) with the points and the epochs at which
// each entry was inserted (ins) and erased (era).
struct Run {
  uint64_t* keys = nullptr;
  uint32_t* ids = nullptr;
  double* xy = nullptr;
  uint32_t* ins = nullptr;
  uint32_t* era = nullptr;
  uint64_t* cells = nullptr;   // grid cells of the points (pack_cell2) if kept (may be null)
};
// Merges the stored run (n entries) with a sorted batch (k entries, local
// ids bids) into `out` (n + k entries).  The batch's entries are inserted at
// `epoch`; with run_off (device, runs + 1 offsets of local ids, run_off[0] =
// 0), those of run r at epoch + r.
hipError_t merge_runs(const Run& stored, uint64_t n, const uint64_t* bkeys, const uint32_t* bids,
                      const double* bxy, uint64_t k, uint32_t id_base, uint32_t epoch,
                      const Run& out, uint64_t* key_of, hipStream_t s,
                      const uint64_t* run_off = nullptr, uint32_t runs = 0);
hipError_t record_keys(const uint64_t* keys, const uint32_t* ids, uint64_t n, uint64_t* key_of,
                       hipStream_t s);
hipError_t erase_entries(const uint32_t* del, uint64_t k, uint32_t next_id, const uint64_t* key_of,
                         const Run& stored, uint64_t n, uint32_t epoch,
                         unsigned long long* erased, hipStream_t s);
// Drops the entries with era <= oldest; *kept_total points at the device
// word that receives the number kept.
size_t compact_entries_scratch(uint64_t n);
hipError_t compact_entries(const Run& stored, uint64_t n, uint32_t oldest, const Run& out,
                           void* scratch, uint64_t** kept_total, hipStream_t s);
hipError_t fill_iota(uint32_t* out, uint64_t k, uint32_t first, hipStream_t s);
// ---- learned index (learned.hip) ----
size_t learned_scratch_bytes();
// Device arrays of a learned index sized for n keys (learned_model_bytes(n)
// bytes, carved by learned_carve).
size_t learned_model_bytes(uint64_t n);
uint32_t learned_max_pieces(uint64_t n);
LearnedArrays learned_carve(void* base, uint64_t n);
// Trains the router (steps Adam steps, 0 = quantile initialisation only) on
// samples of the sorted keys, tabulates it, then fits the leaves' pieces.
// params: kParams floats; losses: 2 floats (sample loss before / after).
hipError_t learned_fit(const uint64_t* keys, uint64_t n, uint32_t steps, float lr, float* params,
                       const LearnedArrays& a, void* scratch, float* losses, hipStream_t s);
// Refits the leaves' pieces for changed keys with the router kept (after an
// update); a must have been carved for at least n keys.
hipError_t learned_refit_leaves(const uint64_t* keys, uint64_t n, const LearnedArrays& a,
                                hipStream_t s);
// Leaf of each key by evaluating the router and through its tabulation.
hipError_t learned_route_both(const float* params, const LearnedArrays& a, const uint64_t* keys,
                              uint64_t count, uint32_t* direct, uint32_t* table, hipStream_t s);
// Gradient of one batch (cnt <= 128 samples) with the trainer's own code.
hipError_t learned_grad(const float* params, const float* xs, const float* ts, int cnt,
                        float* grad, float* loss, hipStream_t s);

}  // namespace sfc
