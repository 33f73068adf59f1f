// Batched distance queries (Alg. 1 over cells(Q); Problem Statement).
//
//   ranges_search  one lane per (query, slot), four slots per query.  Every
//                  lane of a query derives the widened integer box, the
//                  level l = ceil(log2 side), the at most four level-l cells
//                  meeting the box and their merged key intervals (the
//                  Observation gives each cell's interval); slot r then runs
//                  the two searches of interval r over the sorted keys
//                  (binary search or the learned index), optionally split
//                  once into the cell's children that meet the box.  It also
//                  writes what the test needs of each query (a record) and
//                  each workgroup's candidate rows.
//   cells_pack     with early termination: the cells whose quadtree node
//                  holds a point, as a dense (query, cell) work list, so the
//                  search spends lanes only on them.
//   batch_scan     the workgroups' rows -> their first rows, and the batch's
//                  counters (small batches: inside expand_rows).
//   expand_rows    rows -> (slot, first candidate) tiles, and every query's
//                  first row.
//   compact_test   a wave tests 32 rows of 32 candidates each with the exact
//                  distance test, two rows at a time: a hit mask per row, the
//                  hits before it among the 32, and the 32 rows' hits, which
//                  are scanned on the device.
//   compact_write  the same tiles again: the ids of the hits at the scanned
//                  positions, in candidate order; and the CSR offset of every
//                  query, from its first row.
//
// A small batch is four launches: no counter is read by the host, scans are done
// inside the kernels that need them, no memory is cleared, and the last kernel
// stores the counters to host memory (16 queries over 2^16 points: 140 -> 39 us,
// most of it the launches' own latency).
//
// A large batch's search takes its queries in curve order, and with many rows a
// query the rows follow that order too: consecutive tiles then read the same
// lines of the cells and ids and find them in the L2 of their XCD.  The reports
// still leave in query order: the hits of every query (from the rows' prefixes)
// are scanned in query order, and each row is written at its query's offset.
#include <hip/hip_runtime.h>

#include <atomic>

#include <cstdlib>
#include <type_traits>
#include <utility>

#include "common.h"
#include "curve.h"
#include "internal.h"
#include "learned.h"
#include "stree.h"
#include "query_lane.h"

namespace sfc {

namespace {

// ---- what the test pass needs of a query ------------------------------------
//
// A point p with grid cell u = floor(p * S) (S = 2^32 in the plane, 2^21 in
// three dimensions) lies in [u, u + 1) quanta on each axis.  Measured in
// quanta from the query's own cell c = floor(q S), its offset on an axis is
// o = e + th with the integer e = u - c and |th| < 1, so o^2 lies within
// 2|e| + 1 of e^2.  A candidate comes from the query's own cells, which meet
// the box widened by one quantum, so |e| <= E = 6R + 10 with R = d S (exact
// scalings): the sum of the squared offsets lies within the slack
// s = DIM (2E + 1) of the sum of the e^2.  For the Euclidean test:
//   * if sum e^2 <= R^2 (1 - 2^-16) - s, the rounded binary64 test accepts p;
//   * if sum e^2 > R^2 (1 + 2^-16) + s, it rejects p;
// for the square window, |e| <= R (1 - 2^-16) - 1 on every axis accepts and
// |e| > R (1 + 2^-16) + 1 on some axis rejects.  Evaluated in binary32
// (relative errors below 2^-20 all told) these verdicts equal the exact
// test's, whose own rounding is a few 2^-53 relative, when R >= 16 (so the
// slack is small beside R^2).  Other points read their coordinates and take
// the exact test.  A query uses the filter when R >= 16 and its cell lies
// within 2^30 quanta of the domain.  Above R = 2^28 (plane) / 2^17 (three
// dimensions) the cells are compared 2^k quanta wide (u >> k against
// floor(q S 2^-k), k the smallest shift that brings R 2^-k to that limit,
// at most 24): the same bounds hold there with R 2^-k for R, since the
// shifted offsets again differ from the exact ones by less than one.  Then
// |e| < 2^31, exact in 32-bit arithmetic.  Cells sit in one word: x | y << 32,
// or x | y << 21 | z << 42.
struct QueryFilter {
  float acc, rej;   // limits on sum e^2 (or per-axis |e|); filter off: acc = not a number
                    // and rej = +inf, so that neither comparison decides a candidate
  uint32_t minus[3];   // minus the query's cell per axis (low 32 bits), 2^shift quanta wide
  uint32_t shift;   // cells are compared 2^shift quanta wide
  uint32_t pad[2];
};
// The record of a batch whose test reads every candidate's point.
struct QueryExact2 {
  double x, y, d;
  uint32_t pad;
  uint32_t epoch;   // the epoch it is answered at
};
struct QueryExact3 {
  double x, y, z, d;
};
static_assert(sizeof(QueryFilter) == 32 && sizeof(QueryExact2) == 32 && sizeof(QueryExact3) == 32,
              "a record is 32 bytes");

template <int DIM>
constexpr double grid_side() { return DIM == 2 ? 4294967296.0 : 2097152.0; }
// The largest radius, in quanta, compared in whole quanta.
template <int DIM>
constexpr double filter_limit() { return DIM == 2 ? 0x1p28 : 0x1p17; }

template <int DIM>
__device__ __forceinline__ QueryFilter query_filter(const double (&q)[DIM], double d,
                                                    bool window) {
  constexpr double S = grid_side<DIM>(), kMaxR = filter_limit<DIM>();
  const double R0 = d * S;
  int k = 0;
  while (k < 24 && R0 > kMaxR * __builtin_ldexp(1.0, k)) ++k;
  const double R = __builtin_ldexp(R0, -k);   // exact
  bool on = R0 >= 16.0 && R <= kMaxR;
  QueryFilter f{};
  f.shift = (uint32_t)k;
#pragma unroll
  for (int a = 0; a < DIM; ++a) {
    const double qs = q[a] * S;
    on = on && qs > -0x1p30 && qs < S + 0x1p30;
    f.minus[a] = 0u - (uint32_t)(int64_t)__builtin_floor(on ? __builtin_ldexp(qs, -k) : 0.0);
  }
  if (window) {
    f.acc = (float)(R * (1.0 - 0x1p-16) - 1.0);
    f.rej = (float)(R * (1.0 + 0x1p-16) + 1.0);
  } else {
    const double slack = DIM * (2.0 * (6.0 * R + 10.0) + 1.0);
    f.acc = (float)(R * R * (1.0 - 0x1p-16) - slack);
    f.rej = (float)(R * R * (1.0 + 0x1p-16) + slack);
  }
  if (!on) {   // undecided for every candidate: the exact test decides
    f.acc = __uint_as_float(0xFFFFFFFFu);
    f.rej = __builtin_inff();
    f.shift = 0;
  }
  return f;
}

// Writes the record of query j.
template <int DIM>
__device__ __forceinline__ void put_record(const RecordPlan& R, uint64_t j,
                                           const double (&q)[DIM], double d) {
  if (R.mode == kRecordFilter) {
    ((QueryFilter*)R.rec)[j] = query_filter<DIM>(q, d, R.window);
  } else if (R.mode == kRecordExact) {
    if constexpr (DIM == 2)
      ((QueryExact2*)R.rec)[j] = QueryExact2{q[0], q[1], d, 0, R.qepoch ? R.qepoch[j] : R.epoch};
    else
      ((QueryExact3*)R.rec)[j] = QueryExact3{q[0], q[1], q[2], d};
  }
}

// A workgroup's candidates and flags in one word (a workgroup's at most 64
// queries have fewer than 2^39 candidates).
constexpr int kStatShift = 48;
constexpr uint64_t kStatInvalid = 1ull << kStatShift;         // an invalid query
constexpr uint64_t kStatCoarse = 1ull << (kStatShift + 1);    // a radius past the filter limit

// Candidates are processed in rows of 32 (the last of a range partly filled);
// the batch's row count, which capacities refer to, counts rows of 64, of which
// a range has at least half as many.
constexpr int kRowShift = 5;
__device__ __forceinline__ uint64_t rows_of(uint64_t count) {
  return (count + (1u << kRowShift) - 1) >> kRowShift;
}
__device__ __forceinline__ uint64_t rows64_of(uint64_t count) { return (count + 63) >> 6; }

// Every lane's word as the lane permutation CTRL gives it (0 where it has no lane).
template <int CTRL>
__device__ __forceinline__ uint32_t permute_lanes(uint32_t v) {
  uint32_t x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
  asm("" : "+v"(x));   // (a register of its own, never an operand modifier: see bcast16)
  return x;
}
// The value of the lane whose number differs in the bits of X (1..7) from this
// one's; the lanes of a query are active together.
template <int X>
__device__ __forceinline__ uint64_t across(uint64_t v) {
  constexpr int kQuad[4] = {0xE4, 0xB1, 0x4E, 0x1B};   // lanes of four exchanged by xor
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  constexpr int kIn = X & 4 ? X ^ 7 : X;   // mirrored in eight: xor 7
  if constexpr (X & 4) {
    lo = permute_lanes<0x141>(lo);
    hi = permute_lanes<0x141>(hi);
  }
  if constexpr (kIn != 0) {
    lo = permute_lanes<kQuad[kIn]>(lo);
    hi = permute_lanes<kQuad[kIn]>(hi);
  }
  return (uint64_t)hi << 32 | lo;
}
// 1 if the key of that lane comes before this lane's (equal keys by lane).
template <int X>
__device__ __forceinline__ uint32_t before(uint64_t key, int lane) {
  return comes_before<X>(key, across<X>(key), lane);
}
// The lanes of this lane's query (four, bit r for lane r) for which p holds.
__device__ __forceinline__ uint32_t quad_ballot(bool p) {
  return (uint32_t)(__ballot(p) >> (lane_id() & ~3u)) & 15u;
}

// One lane per (query, slot): four slots per query (the method's ranges),
// or eight (REFINE: two runs per cell of cells(Q)).  QUAD: the lane's work is the
// body in query_quad.inc (its own cell alone; the query's four lanes exchange keys
// to order and merge them); else (early termination's list, inspected ranges) the
// one in query_lane.inc.  perm non-null: the queries in curve order, so that
// the searches of a workgroup meet in the same lines of the key array; slots
// and records are laid out by query.  Each workgroup (64 queries) also sums
// its counters, and its candidate rows if it holds 64 consecutive queries: one
// word each per workgroup, no atomics (those of every workgroup on one address
// serialise across the XCDs), and nothing to clear beforehand.
// At least five waves per SIMD (at most 102 registers): the chains of
// dependent probes need waves in flight.
template <int CURVE, bool REFINE, int SEARCH, bool QUAD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void ranges_search(
    const double2* __restrict__ q, const double* __restrict__ delta, uint64_t m,
    const uint64_t* __restrict__ keys, uint64_t n, LearnedView lv, StreeView sv,
    uint32_t refine_min, bool ball, const uint32_t* __restrict__ occ,
    const uint64_t* __restrict__ pairs, const uint32_t* __restrict__ pair_total,
    const uint32_t* __restrict__ qset, const uint64_t* __restrict__ set_off, uint32_t n_sets,
    const uint32_t* __restrict__ perm, RecordPlan record, uint2* __restrict__ slots,
    uint64_t* __restrict__ blk_rows, uint64_t* __restrict__ blk_stat,
    uint64_t* __restrict__ blk_rows64, uint32_t* __restrict__ blk_learned,
    uint64_t* __restrict__ dbg_lo,
    uint64_t* __restrict__ dbg_hi, uint64_t* __restrict__ dbg_b, uint64_t* __restrict__ dbg_e,
    uint32_t* __restrict__ dbg_nr) {
  constexpr bool LEARNED = SEARCH == 1;
  __shared__ uint16_t lut[CURVE == SFC_CURVE_HILBERT ? 1024 : 1];
  // Workgroups past the listed pairs have nothing to do (uniform per block).
  if (pairs && (uint64_t)blockIdx.x * 256 >= *pair_total) {
    if (threadIdx.x == 0) {
      blk_stat[blockIdx.x] = 0;
      blk_rows64[blockIdx.x] = 0;
      if (LEARNED) blk_learned[blockIdx.x] = 0;
    }
    return;
  }
  if (CURVE == SFC_CURVE_HILBERT)
    for (int i = threadIdx.x; i < 1024; i += 256) lut[i] = kHilbertLutConst.v[i];
  __syncthreads();
  // Lane -> (query, cell): four lanes per query, or (pairs) one lane per
  // cell that survived early termination, packed densely; idle lanes take
  // j = m.
  const uint64_t g = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  const bool act = pairs ? g < *pair_total : (g >> 2) < m;
  const uint64_t pair = pairs ? (act ? pairs[g] : 0) : g;   // 4 * query + cell
  const int r = (int)(pair & 3);
  const uint64_t j = act ? (perm ? perm[pair >> 2] : pair >> 2) : m;
  uint64_t sidx = 4 * j + r;

  uint64_t b0 = 0, e0 = 0, b1 = 0, e1 = 0, klo = 0, khi = 0;
  int nr = 0;
  bool bad = false, coarse = false;
  uint32_t fb = 0, ends = 0, pruned = 0;
  if (!pairs && j < m && r == 0 && record.mode != kRecordNone) {
    const double2 qq = q[j];
    const double c[2] = {qq.x, qq.y}, d = delta[j];
    put_record<2>(record, j, c, d);
    coarse = d * grid_side<2>() > filter_limit<2>();
  }
  // With point sets, a query searches only its own set's keys: positions
  // [base, base + nn) of the sorted arrays.
  uint64_t base = 0, nn = n;
  if (j < m && qset) {
    const uint32_t sj = qset[j];
    if (sj >= n_sets) {
      bad = true;
      nn = 0;
    } else {
      base = set_off[sj];
      nn = set_off[sj + 1] - base;
    }
  }
  if constexpr (QUAD) {
#include "query_quad.inc"
  } else {
#include "query_lane.inc"
    (void)pruned;   // counted where the work list is made
  }
  // Candidates, rows, flags (and learned-index endpoints and fallbacks) of
  // the workgroup.
  __shared__ uint64_t s_cand[4], s_rows[4], s_rows64[4];
  __shared__ uint32_t s_learned[4];
  uint64_t wc = (e0 - b0) + (e1 - b1), wr = rows_of(e0 - b0) + rows_of(e1 - b1);
  uint64_t wr64 = rows64_of(e0 - b0) + rows64_of(e1 - b1);
  uint32_t wl = (ends << 16) | fb;
  const uint64_t flags = (__ballot(bad) != 0 ? kStatInvalid : 0) |
                         (__ballot(coarse) != 0 ? kStatCoarse : 0);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    wc += __shfl_xor(wc, o, 64);
    wr += __shfl_xor(wr, o, 64);
    wr64 += __shfl_xor(wr64, o, 64);
    if (LEARNED) wl += __shfl_xor(wl, o, 64);
  }
  const uint32_t wv = threadIdx.x >> 6;
  if (lane_id() == 0) {
    s_cand[wv] = wc | flags;
    s_rows[wv] = wr;
    s_rows64[wv] = wr64;
    if (LEARNED) s_learned[wv] = wl;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t c = 0, f = 0;
    for (int w = 0; w < 4; ++w) {
      c += s_cand[w] & (kStatInvalid - 1);
      f |= s_cand[w] & ~(kStatInvalid - 1);
    }
    blk_stat[blockIdx.x] = c | f;
    blk_rows64[blockIdx.x] = s_rows64[0] + s_rows64[1] + s_rows64[2] + s_rows64[3];
    if (!pairs) blk_rows[blockIdx.x] = s_rows[0] + s_rows[1] + s_rows[2] + s_rows[3];
    if (LEARNED)
      blk_learned[blockIdx.x] = s_learned[0] + s_learned[1] + s_learned[2] + s_learned[3];
  }
  if (j < m) {
    if (!REFINE) {
      slots[sidx] = make_uint2((uint32_t)b0, (uint32_t)(e0 - b0));
      if (dbg_lo) {
        dbg_lo[sidx] = klo;
        dbg_hi[sidx] = khi;
        dbg_b[sidx] = b0;
        dbg_e[sidx] = e0;
        if (r == 0) dbg_nr[j] = (uint32_t)nr;
      }
    } else {
      ((uint4*)slots)[sidx] =
          make_uint4((uint32_t)b0, (uint32_t)(e0 - b0), (uint32_t)b1, (uint32_t)(e1 - b1));
    }
  }
}

// ---- three dimensions (d = 3 Morton codes) ------------------------------------

constexpr double kTwo22 = 4194304.0;            // 2^22
constexpr double kTwoM29 = 1.0 / 536870912.0;   // 2^-29

// The d = 3 test: the squares summed left to right, no contraction.
__device__ __forceinline__ bool within3(double px, double py, double pz, double qx, double qy,
                                        double qz, double d) {
#pragma clang fp contract(off)
  const double dx = px - qx;
  const double dy = py - qy;
  const double dz = pz - qz;
  const double t = dx * dx;
  const double u = dy * dy;
  const double v = dz * dz;
  const double s = (t + u) + v;
  return s <= d * d;
}

__device__ __forceinline__ bool within_window3(double px, double py, double pz, double qx,
                                               double qy, double qz, double d) {
#pragma clang fp contract(off)
  const double dx = px - qx;
  const double dy = py - qy;
  const double dz = pz - qz;
  return fabs(dx) <= d && fabs(dy) <= d && fabs(dz) <= d;
}

// One axis of the widened box on the 2^21 grid: w = 1 + floor((|c| + d)
// 2^-29) quanta cover the rounding of the test.
__device__ __forceinline__ bool axis_box3(double c, double d, int64_t& lo, int64_t& hi) {
#pragma clang fp contract(off)
  double wr = __builtin_floor((__builtin_fabs(c) + d) * kTwoM29);
  wr = wr > kTwo22 ? kTwo22 : wr;
  const int64_t w = 1 + (int64_t)wr;
  double a = (c - d) * kTwo21, b = (c + d) * kTwo21;
  a = a < -kTwo22 ? -kTwo22 : (a > kTwo22 ? kTwo22 : a);
  b = b < -kTwo22 ? -kTwo22 : (b > kTwo22 ? kTwo22 : b);
  int64_t l = (int64_t)__builtin_floor(a) - w;
  int64_t h = (int64_t)__builtin_floor(b) + w;
  l = l < 0 ? 0 : l;
  h = h > (int64_t)kMaxCell3 ? (int64_t)kMaxCell3 : h;
  lo = l;
  hi = h;
  return l <= h;
}

// Merged key intervals of the level-l cubes meeting the widened box (at most
// 8), ascending and non-adjacent.
__device__ int query_ranges3(double qx, double qy, double qz, double d, uint64_t lo[8],
                             uint64_t hi[8]) {
  int64_t b[6];
  if (!axis_box3(qx, d, b[0], b[1]) || !axis_box3(qy, d, b[2], b[3]) ||
      !axis_box3(qz, d, b[4], b[5]))
    return 0;
  uint64_t side = (uint64_t)(b[1] - b[0] + 1);
  side = (uint64_t)(b[3] - b[2] + 1) > side ? (uint64_t)(b[3] - b[2] + 1) : side;
  side = (uint64_t)(b[5] - b[4] + 1) > side ? (uint64_t)(b[5] - b[4] + 1) : side;
  const int L = side <= 1 ? 0 : 64 - __clzll(side - 1);
  if (L >= 21) {
    lo[0] = 0;
    hi[0] = (1ull << 63) - 1;
    return 1;
  }
  const uint64_t span = (1ull << (3 * L)) - 1;
  int k = 0;
  for (uint32_t cx = (uint32_t)(b[0] >> L); cx <= (uint32_t)(b[1] >> L); ++cx)
    for (uint32_t cy = (uint32_t)(b[2] >> L); cy <= (uint32_t)(b[3] >> L); ++cy)
      for (uint32_t cz = (uint32_t)(b[4] >> L); cz <= (uint32_t)(b[5] >> L); ++cz) {
        const uint64_t key = morton3_key(cx << L, cy << L, cz << L) & ~span;
        int t = k++;
        for (; t > 0 && lo[t - 1] > key; --t) lo[t] = lo[t - 1];
        lo[t] = key;
      }
  int r = 0;
  for (int i = 0; i < k; ++i) {
    if (r > 0 && hi[r - 1] + 1 == lo[i]) {
      hi[r - 1] = lo[i] | span;
    } else {
      lo[r] = lo[i];
      hi[r] = lo[i] | span;
      ++r;
    }
  }
  return r;
}

// One lane per (query, slot): eight slots per query, each a merged interval
// of the query's cubes.  REFINE: one lane per cube (unmerged); a cube
// holding more than refine_min keys is split once, its children that meet
// the box forming at most four runs of consecutive children in key order
// (four slots per cube, 32 per query), each found by two searches inside the
// cube's index range.  The reported ids and their order do not change.
template <int SEARCH, bool REFINE>
// Refined, a lane works out its own cube and its place among the eight lanes'
// (all eight cubes in every lane, sorted by a network of 19 exchanges, took 71
// registers for 54 and a quarter more instructions: 1.00 ms for 0.98 with the
// static search tree, 2^20 queries over 2^24 keys; the lines of memory bound both).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void ranges_search3(
    const double* __restrict__ q, const double* __restrict__ delta, uint64_t m,
    const uint64_t* __restrict__ keys, uint64_t n, LearnedView lv, StreeView sv,
    uint32_t refine_min, const uint32_t* __restrict__ perm, RecordPlan record,
    uint2* __restrict__ slots, uint64_t* __restrict__ blk_rows,
    uint64_t* __restrict__ blk_stat, uint64_t* __restrict__ blk_rows64) {
  const uint64_t g = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  const uint64_t j = (g >> 3) < m ? (perm ? perm[g >> 3] : g >> 3) : m;
  const int r = (int)(g & 7);
  int slot = r;
  uint64_t B[4] = {0, 0, 0, 0}, E[4] = {0, 0, 0, 0};
  uint32_t fb = 0;
  bool bad = false, coarse = false;
  if (j < m) {
    const double qx = q[3 * j], qy = q[3 * j + 1], qz = q[3 * j + 2], d = delta[j];
    if (r == 0) {
      const double c[3] = {qx, qy, qz};
      put_record<3>(record, j, c, d);
      coarse = d * grid_side<3>() > filter_limit<3>();
    }
    if (epoch_rejected(record, j) ||
        !(finite64(qx) && finite64(qy) && finite64(qz) && finite64(d) && d >= 0.0)) {
      bad = true;
    } else if (!REFINE) {
      uint64_t lo[8], hi[8];
      const int nr = query_ranges3(qx, qy, qz, d, lo, hi);
      // The lane's range, taken with static indexes (a runtime index into
      // the arrays would put them in scratch memory).
      uint64_t mlo = 0, mhi = 0;
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (c == r) {
          mlo = lo[c];
          mhi = hi[c];
        }
      if (r < nr) find_range<SEARCH>(keys, n, lv, sv, mlo, mhi, B[0], E[0], fb);
    } else {
      // A box of side at most 2^L meets at most two level-L cells per axis:
      // lane r takes the cube at offsets (r, r / 2, r / 4) mod 2, and its slot
      // is its key's place among the eight lanes' (those without a cube last).
      int64_t b[6] = {0, -1, 0, -1, 0, -1};
      const bool some = axis_box3(qx, d, b[0], b[1]) && axis_box3(qy, d, b[2], b[3]) &&
                        axis_box3(qz, d, b[4], b[5]);
      uint64_t side = (uint64_t)(b[1] - b[0] + 1);
      side = (uint64_t)(b[3] - b[2] + 1) > side ? (uint64_t)(b[3] - b[2] + 1) : side;
      side = (uint64_t)(b[5] - b[4] + 1) > side ? (uint64_t)(b[5] - b[4] + 1) : side;
      const int L = side <= 1 ? 0 : 64 - __clzll(side - 1) < 21 ? 64 - __clzll(side - 1) : 21;
      const uint32_t mx = (uint32_t)(b[0] >> L) + (r & 1);
      const uint32_t my = (uint32_t)(b[2] >> L) + ((r >> 1) & 1);
      const uint32_t mz = (uint32_t)(b[4] >> L) + (r >> 2);
      const bool in = some && mx <= (uint32_t)(b[1] >> L) && my <= (uint32_t)(b[3] >> L) &&
                      mz <= (uint32_t)(b[5] >> L);
      const uint64_t key = morton3_key(mx << L, my << L, mz << L);
      const uint64_t mlo = in ? key : ~0ull;
      slot = (int)(before<1>(mlo, r) + before<2>(mlo, r) + before<3>(mlo, r) + before<4>(mlo, r) +
                   before<5>(mlo, r) + before<6>(mlo, r) + before<7>(mlo, r));
      if (in) {
        const uint64_t span = L >= 21 ? (1ull << 63) - 1 : (1ull << (3 * L)) - 1;
        find_range<SEARCH>(keys, n, lv, sv, mlo, mlo | span, B[0], E[0], fb);
        if (E[0] - B[0] > refine_min && L >= 1 && L < 21) {
          const int Lc = L - 1;
          const uint64_t cspan = (1ull << (3 * Lc)) - 1;
          const int64_t hs = (int64_t)1 << Lc;
          uint32_t meet = 0;   // bit c: child c (x + 2y + 4z) meets the box
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            const int64_t x0 = (int64_t)(2 * mx + (c & 1)) << Lc;
            const int64_t y0 = (int64_t)(2 * my + ((c >> 1) & 1)) << Lc;
            const int64_t z0 = (int64_t)(2 * mz + (c >> 2)) << Lc;
            const bool in = x0 <= b[1] && x0 + hs - 1 >= b[0] && y0 <= b[3] &&
                            y0 + hs - 1 >= b[2] && z0 <= b[5] && z0 + hs - 1 >= b[4];
            meet |= (uint32_t)in << c;
          }
          if (meet != 0xFFu) {
            // Runs of consecutive children: the k-th run starts at the k-th
            // set bit of `st` and ends at the k-th set bit of `en`.
            // The runs lie in the cube's index range: searched there, one
            // after the other (four runs in lockstep took longer).
            const uint64_t pb = B[0], pe = E[0];
            uint32_t st = meet & ~(meet << 1);
            uint32_t en = meet & ~(meet >> 1);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              B[k] = E[k] = 0;
              if (st) {
                const int c0 = __builtin_ctz(st), c1 = __builtin_ctz(en);
                st &= st - 1;
                en &= en - 1;
                const uint64_t klo = mlo | ((uint64_t)c0 << (3 * Lc));
                const uint64_t khi = mlo | ((uint64_t)c1 << (3 * Lc)) | cspan;
                uint64_t x, y;
                search_pair(keys + pb, pe - pb, klo, khi, x, y);
                B[k] = pb + x;
                E[k] = pb + y;
              }
            }
          }
        }
      }
    }
  }
  // Candidates, rows and flags of the workgroup (32 queries).
  __shared__ uint64_t s_cand[4], s_rows[4], s_rows64[4];
  uint64_t wc = 0, wr = 0, wr64 = 0;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    wc += E[t] - B[t];
    wr += rows_of(E[t] - B[t]);
    wr64 += rows64_of(E[t] - B[t]);
  }
  const uint64_t flags = (__ballot(bad) != 0 ? kStatInvalid : 0) |
                         (__ballot(coarse) != 0 ? kStatCoarse : 0);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    wc += __shfl_xor(wc, o, 64);
    wr += __shfl_xor(wr, o, 64);
    wr64 += __shfl_xor(wr64, o, 64);
  }
  if (lane_id() == 0) {
    s_cand[threadIdx.x >> 6] = wc | flags;
    s_rows[threadIdx.x >> 6] = wr;
    s_rows64[threadIdx.x >> 6] = wr64;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t c = 0, f = 0;
    for (int w = 0; w < 4; ++w) {
      c += s_cand[w] & (kStatInvalid - 1);
      f |= s_cand[w] & ~(kStatInvalid - 1);
    }
    blk_stat[blockIdx.x] = c | f;
    blk_rows64[blockIdx.x] = s_rows64[0] + s_rows64[1] + s_rows64[2] + s_rows64[3];
    blk_rows[blockIdx.x] = s_rows[0] + s_rows[1] + s_rows[2] + s_rows[3];
  }
  if (j < m) {
    const uint64_t sidx = 8 * j + slot;
    if (!REFINE) {
      slots[sidx] = make_uint2((uint32_t)B[0], (uint32_t)(E[0] - B[0]));
    } else {
      uint4* o = (uint4*)(slots + 4 * sidx);
#pragma unroll
      for (int t = 0; t < 4; t += 2)
        o[t / 2] = make_uint4((uint32_t)B[t], (uint32_t)(E[t] - B[t]), (uint32_t)B[t + 1],
                              (uint32_t)(E[t + 1] - B[t + 1]));
    }
  }
}

// Early termination: whether many cells of a batch's queries hold points, from a
// sample of 1024 of them (*wanted = 1 or 0).  One workgroup.
constexpr uint32_t kSampled = 1024;
template <int CURVE>
__global__ __launch_bounds__(kSampled) void sample_cells(const double2* __restrict__ q,
                                                         const double* __restrict__ delta,
                                                         uint64_t m,
                                                         const uint32_t* __restrict__ occ,
                                                         uint32_t least, uint32_t* wanted) {
  __shared__ uint16_t lut[CURVE == SFC_CURVE_HILBERT ? 1024 : 1];
  __shared__ uint32_t s_sum[kSampled / kWave];
  const uint32_t tid = threadIdx.x;
  if (CURVE == SFC_CURVE_HILBERT) lut[tid] = kHilbertLutConst.v[tid];
  __syncthreads();
  const uint64_t j = tid * m / kSampled;
  const double2 qq = q[j];
  const double d = delta[j];
  uint32_t sum = 0;
  if (finite64(qq.x) && finite64(qq.y) && finite64(d) && d >= 0.0) {
    uint64_t lo[4], hi[4];
    uint32_t cx[4], cy[4], pr = 0;
    int64_t box[4];
    int L = 0;
    sum = (uint32_t)query_cells<CURVE>(lut, qq.x, qq.y, d, lo, hi, cx, cy, &L, box, occ, &pr);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (lane_id() == 0) s_sum[tid >> 6] = sum;
  __syncthreads();
  if (tid == 0) {
    for (uint32_t w = 1; w < kSampled / kWave; ++w) sum += s_sum[w];
    *wanted = sum >= least ? 1u : 0u;
  }
}

// The cells of every query that survive early termination, as (query, cell)
// pairs (4 * query + cell) for the search.  One
// thread per query; block b lists its pairs at the start of its own region
// pairs[1024 b ..] and its counts of pairs and of pruned cells in blk_cnt[b]
// and blk_pruned[b] (pack_scan and pack_move then make the list dense, in
// query order), its flags in blk_flags[b].  No atomic on a shared word:
// one per block, from every block of the grid, serialises across the XCDs.
// The query's slots are cleared and its record is written here; invalid
// queries (and epochs) raise the flag and list no cell.  perm (may be null): the
// queries in the order to list them in (if *wanted, wanted given).
template <int CURVE, bool REFINE>
__global__ __launch_bounds__(256) void cells_pack(
    const double2* __restrict__ q, const double* __restrict__ delta, uint64_t m,
    const uint32_t* __restrict__ occ, uint64_t* __restrict__ pairs,
    uint32_t* __restrict__ blk_cnt, uint32_t* __restrict__ blk_pruned,
    uint64_t* __restrict__ blk_flags, RecordPlan record, uint2* __restrict__ slots,
    const uint32_t* __restrict__ perm, const uint32_t* wanted) {
  __shared__ uint16_t lut[CURVE == SFC_CURVE_HILBERT ? 1024 : 1];
  __shared__ uint32_t s_cnt[4];
  __shared__ uint32_t s_pr[4];
  __shared__ uint64_t s_fl[4];
  if (CURVE == SFC_CURVE_HILBERT)
    for (int i = threadIdx.x; i < 1024; i += 256) lut[i] = kHilbertLutConst.v[i];
  __syncthreads();
  const uint64_t at = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  const uint64_t j = perm && at < m && (!wanted || *wanted) ? perm[at] : at;
  uint32_t nr = 0, pr = 0;
  bool bad = false, coarse = false;
  if (j < m) {
    const double2 qq = q[j];
    const double d = delta[j];
    const double c[2] = {qq.x, qq.y};
    put_record<2>(record, j, c, d);
    coarse = d * grid_side<2>() > filter_limit<2>();
    if (epoch_rejected(record, j) ||
        !(finite64(qq.x) && finite64(qq.y) && finite64(d) && d >= 0.0)) {
      bad = true;
    } else if (REFINE) {
      uint64_t lo[4], hi[4];
      uint32_t cx[4], cy[4];
      int64_t box[4];
      int L = 0;
      nr = (uint32_t)query_cells<CURVE>(lut, qq.x, qq.y, d, lo, hi, cx, cy, &L, box, occ, &pr);
    } else {
      uint64_t lo[4], hi[4];
      nr = (uint32_t)query_ranges<CURVE>(lut, qq.x, qq.y, d, lo, hi, occ, &pr);
    }
    // Every slot of the query starts empty; the search then writes the slots
    // of the listed cells.
    uint4* sl = (uint4*)(slots + (REFINE ? 8 : 4) * j);
#pragma unroll
    for (int i = 0; i < (REFINE ? 4 : 2); ++i) sl[i] = make_uint4(0, 0, 0, 0);
  }
  const uint64_t flags = (__ballot(bad) != 0 ? kStatInvalid : 0) |
                         (__ballot(coarse) != 0 ? kStatCoarse : 0);
  // Block-exclusive offsets of the cell counts: wave prefix, then waves.
  const uint32_t lane = lane_id(), wv = threadIdx.x >> 6;
  uint32_t inc = nr, wp = pr;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(inc, o, 64);
    if (lane >= (uint32_t)o) inc += t;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) wp += __shfl_xor(wp, o, 64);
  if (lane == 63) s_cnt[wv] = inc;
  if (lane == 0) {
    s_pr[wv] = wp;
    s_fl[wv] = flags;
  }
  __syncthreads();
  uint32_t before = 0;
  for (uint32_t w = 0; w < wv; ++w) before += s_cnt[w];
  if (threadIdx.x == 0) {
    blk_cnt[blockIdx.x] = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
    blk_pruned[blockIdx.x] = s_pr[0] + s_pr[1] + s_pr[2] + s_pr[3];
    blk_flags[blockIdx.x] = s_fl[0] | s_fl[1] | s_fl[2] | s_fl[3];
  }
  const uint64_t o = (uint64_t)blockIdx.x * 1024 + before + inc - nr;
  for (uint32_t r = 0; r < nr; ++r) pairs[o + r] = 4 * j + r;
}

// One workgroup: the exclusive scan of the blocks' pair counts (blk_pre, and
// the list's length in *pair_total).
__global__ __launch_bounds__(1024) void pack_scan(const uint32_t* __restrict__ blk_cnt,
                                                  uint32_t nblk, uint32_t* __restrict__ blk_pre,
                                                  uint32_t* pair_total) {
  __shared__ uint32_t s_w[16];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  uint32_t carry = 0;
  for (uint32_t b0 = 0; b0 < nblk; b0 += 1024) {
    const uint32_t b = b0 + tid;
    const uint32_t v = b < nblk ? blk_cnt[b] : 0u;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (lane >= (uint32_t)o) x += y;
    }
    if (lane == 63) s_w[wv] = x;
    __syncthreads();
    uint32_t before = carry;
    for (uint32_t w = 0; w < wv; ++w) before += s_w[w];
    if (b < nblk) blk_pre[b] = before + x - v;
    uint32_t all = 0;
    for (uint32_t w = 0; w < 16; ++w) all += s_w[w];
    carry += all;
    __syncthreads();
  }
  if (tid == 0) *pair_total = carry;
}

// Block b moves its region's pairs to their place in the dense list.
__global__ __launch_bounds__(256) void pack_move(const uint64_t* __restrict__ pairs_in,
                                                 const uint32_t* __restrict__ blk_cnt,
                                                 const uint32_t* __restrict__ blk_pre,
                                                 uint64_t* __restrict__ pairs_out) {
  const uint32_t c = blk_cnt[blockIdx.x], at = blk_pre[blockIdx.x];
  for (uint32_t i = threadIdx.x; i < c; i += 256)
    pairs_out[at + i] = pairs_in[(uint64_t)blockIdx.x * 1024 + i];
}

// The candidates are laid out in rows of 32: each query slot (segment) s
// owns rows [row_off[s], row_off[s+1]), row k of s holding its candidates
// 32k .. 32k+31 (the last row partly filled).  So every row belongs to one slot
// and one query.  A wave takes two rows at a time (short ranges are the rule:
// 19 candidates a range for 10 reports aimed at, so that a row of 64 would leave
// two lanes of three idle), 32 rows in all, its unit; a tile is four waves' rows.
constexpr uint32_t kUnitRows = 32;
constexpr int kUnitShift = 5;
constexpr int kUnitSteps = 16;                         // pairs of rows
constexpr uint32_t kTileUnits = 4;
constexpr uint64_t kTileRows = kTileUnits * kUnitRows; // rows of 32
static_assert(kTileRows == 2 * kCompactTileRows, "a tile holds 64 rows of 64 candidates");

// Tiles of a chunk's rows [rbase, row_end); none of a batch that is not tested.
__device__ __forceinline__ uint64_t chunk_tiles(uint64_t total_all, uint64_t rbase,
                                                uint64_t row_end, bool over) {
  if (over) return 0;
  const uint64_t total = total_all < row_end ? total_all : row_end;
  return total > rbase ? (total - rbase + kTileRows - 1) / kTileRows : 0;
}

// Tile of step i of workgroup b of a grid of a multiple of eight workgroups,
// ~0 past the last: each XCD (the hardware deals workgroups to the eight XCDs
// in turn) takes a contiguous range of the tiles, so that the lines that
// consecutive tiles share are fetched into one L2.
__device__ __forceinline__ uint64_t xcd_tile(uint64_t b, uint64_t grid, uint64_t i,
                                             uint64_t ntiles) {
  const uint64_t per = (ntiles + 7) / 8;
  const uint64_t k = (b >> 3) + i * (grid >> 3);
  const uint64_t t = (b & 7) * per + k;
  return k < per && t < ntiles ? t : ~0ull;
}

// Exclusive scan of one uint64 per thread over 256 threads; *total gets the
// sum.
__device__ __forceinline__ uint64_t scan256_u64(uint64_t v, uint64_t* s_w, uint64_t* total) {
  const uint32_t lane = lane_id(), wv = threadIdx.x >> 6;
  uint64_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(x, o, 64);
    if (lane >= (uint32_t)o) x += y;
  }
  if (lane == 63) s_w[wv] = x;
  __syncthreads();
  uint64_t before = 0;
  for (uint32_t w = 0; w < wv; ++w) before += s_w[w];
  *total = s_w[0] + s_w[1] + s_w[2] + s_w[3];
  __syncthreads();
  return before + x - v;
}

// The batch's counters, from those of the workgroups: stat and rows64 (ns words
// each: candidates and flags; rows of 64), learned (ns words or null: endpoints << 16 |
// fallbacks), and with early termination flags and pruned (np words each, or
// null).  Every thread of the workgroup calls it; thread 0 holds the result.
struct BatchStats {
  const uint64_t* stat;
  const uint64_t* rows64;
  const uint32_t* learned;
  uint32_t ns;
  const uint64_t* flags;
  const uint32_t* pruned;
  uint32_t np;
};

// Adds the counters of entries [first, ns) in steps of `step` (np likewise) to v:
// candidates, endpoints, fallbacks, pruned, rows, flags.
__device__ __forceinline__ void add_stats(const BatchStats& B, uint32_t first, uint32_t step,
                                          uint32_t ns, uint32_t np, uint64_t (&v)[6]) {
  // Eight words in flight per thread: those past the end load the last one
  // and are not added.
  for (uint32_t i0 = first; i0 < ns; i0 += step * 8) {
    uint64_t w[8], rw[8];
    uint32_t l[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      const uint32_t i = i0 + k * step, ic = i < ns ? i : ns - 1;
      w[k] = B.stat[ic];
      rw[k] = B.rows64[ic];
      l[k] = B.learned ? B.learned[ic] : 0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k)
      if (i0 + k * step < ns) {
        v[0] += w[k] & (kStatInvalid - 1);
        v[5] |= w[k] >> kStatShift;
        v[4] += rw[k];
        v[1] += l[k] >> 16;
        v[2] += l[k] & 0xFFFFu;
      }
  }
  for (uint32_t i = first; i < np; i += step) {
    v[3] += B.pruned[i];
    v[5] |= B.flags[i] >> kStatShift;
  }
}

// The workgroup's sums of v, in thread 0.
template <int WAVES>
__device__ __forceinline__ void sum_over_waves(uint64_t (&v)[6]) {
  __shared__ uint64_t s_v[6][WAVES];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
#pragma unroll
    for (int k = 0; k < 5; ++k) v[k] += __shfl_xor(v[k], o, 64);
    v[5] |= __shfl_xor(v[5], o, 64);
  }
  if (lane_id() == 0)
#pragma unroll
    for (int k = 0; k < 6; ++k) s_v[k][threadIdx.x >> 6] = v[k];
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < WAVES; ++w) {
#pragma unroll
      for (int k = 0; k < 5; ++k) v[k] += s_v[k][w];
      v[5] |= s_v[5][w];
    }
}

__device__ __forceinline__ void put_stats(const uint64_t (&v)[6], BatchStatus* status,
                                          BatchStatus* host) {
  BatchStatus st{};
  st.candidates = v[0];
  st.endpoints = v[1];
  st.fallbacks = v[2];
  st.pruned = v[3];
  st.rows = v[4];
  if (v[5] & 1) st.err |= kErrInvalidQuery;
  if (v[5] & 2) st.coarse = 1;
  *status = st;
  if (host) *host = st;
}

// The same by one workgroup alone.
template <int WAVES>
__device__ __forceinline__ void sum_stats(const BatchStats& B, BatchStatus* status,
                                          BatchStatus* host) {
  uint64_t v[6] = {0, 0, 0, 0, 0, 0};
  add_stats(B, threadIdx.x, WAVES * 64, B.ns, B.np, v);
  sum_over_waves<WAVES>(v);
  if (threadIdx.x == 0) put_stats(v, status, host);
}

// Batches of more search workgroups than this sum their rows and counters in two
// launches: group_sums by groups of kGroupBlocks, then one workgroup over the
// groups.  (One workgroup over all is a chain of rounds of loads: 83 us at 2^16
// workgroups and 21 at 2^14, by groups 12 and 9; at 2^12 both take about 9.)
constexpr uint32_t kOneScan = 4096;
constexpr uint32_t kGroupBlocks = 1024;
struct GroupSums {
  uint64_t rows;     // of the group; then of the groups before it
  uint64_t v[6];     // the counters of its entries
  uint64_t pad;
};

// Group g: its rows and counters, and the exclusive scan of its workgroups' rows.
__global__ __launch_bounds__(256) void group_sums(const uint64_t* __restrict__ blk_rows,
                                                  uint32_t nblk, uint64_t* __restrict__ blk_off,
                                                  BatchStats B, bool stats,
                                                  GroupSums* __restrict__ groups) {
  __shared__ uint64_t s_w[4];
  const uint32_t first = blockIdx.x * kGroupBlocks, tid = threadIdx.x;
  constexpr uint32_t kPer = kGroupBlocks / 256;
  const uint32_t f = first + tid * kPer;
  uint64_t v[kPer], sum = 0, total;
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) v[i] = f + i < nblk ? blk_rows[f + i] : 0;
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) sum += v[i];
  uint64_t run = scan256_u64(sum, s_w, &total);
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    if (f + i < nblk) blk_off[f + i] = run;
    run += v[i];
  }
  uint64_t c[6] = {0, 0, 0, 0, 0, 0};
  if (stats) {
    const uint32_t end = first + kGroupBlocks;
    add_stats(B, first + tid, 256, B.ns < end ? B.ns : end, B.np < end ? B.np : end, c);
    sum_over_waves<4>(c);
  }
  if (tid == 0) {
    groups[blockIdx.x].rows = total;
#pragma unroll
    for (int k = 0; k < 6; ++k) groups[blockIdx.x].v[k] = c[k];
  }
}

// One workgroup: the groups' rows -> the rows before each; the total and the
// counters as batch_scan gives them.
__global__ __launch_bounds__(256) void group_scan(GroupSums* __restrict__ groups, uint32_t count,
                                                  uint64_t* __restrict__ rows_out, bool stats,
                                                  BatchStatus* status, BatchStatus* host) {
  __shared__ uint64_t s_w[4];
  const uint32_t tid = threadIdx.x;
  uint64_t carry = 0, c[6] = {0, 0, 0, 0, 0, 0};
  for (uint32_t g0 = 0; g0 < count; g0 += 256) {
    const uint32_t g = g0 + tid;
    uint64_t rows = 0, total;
    if (g < count) {
      rows = groups[g].rows;
#pragma unroll
      for (int k = 0; k < 5; ++k) c[k] += groups[g].v[k];
      c[5] |= groups[g].v[5];
    }
    const uint64_t before = scan256_u64(rows, s_w, &total);
    if (g < count) groups[g].rows = carry + before;
    carry += total;
  }
  if (tid == 0) *rows_out = carry;
  if (stats) {
    sum_over_waves<4>(c);
    if (tid == 0) put_stats(c, status, host);
  }
}

// One workgroup: the exclusive scan of the workgroups' rows (blk_off, the
// total in *rows_out), and the batch's counters in *status (and *host, host
// memory, if not null); stats false: the counters stay.
__global__ __launch_bounds__(1024) void batch_scan(const uint64_t* __restrict__ blk_rows,
                                                   uint32_t nblk, uint64_t* __restrict__ blk_off,
                                                   uint64_t* __restrict__ rows_out,
                                                   BatchStats B, bool stats, BatchStatus* status,
                                                   BatchStatus* host) {
  constexpr uint32_t kPer = 8;
  __shared__ uint64_t s_w[16];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  uint64_t carry = 0;
  for (uint32_t b0 = 0; b0 < nblk; b0 += 1024 * kPer) {
    const uint32_t f = b0 + tid * kPer;
    uint64_t v[kPer], sum = 0;
    // Every load in flight at once: entries past the end load the last one
    // and count as zero.
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) v[i] = blk_rows[f + i < nblk ? f + i : nblk - 1];
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      if (f + i >= nblk) v[i] = 0;
      sum += v[i];
    }
    uint64_t x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t y = __shfl_up(x, o, 64);
      if (lane >= (uint32_t)o) x += y;
    }
    if (lane == 63) s_w[wv] = x;
    __syncthreads();
    uint64_t run = carry + x - sum, all = 0;
    for (uint32_t w = 0; w < 16; ++w) {
      if (w < wv) run += s_w[w];
      all += s_w[w];
    }
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      if (f + i < nblk) blk_off[f + i] = run;
      run += v[i];
    }
    carry += all;
    __syncthreads();
  }
  if (tid == 0) *rows_out = carry;
  if (stats) sum_stats<16>(B, status, host);
}

// The K consecutive slots from `first` on, in the order of the places (perm:
// the query of each, 2^ss slots; null: the queries' own), empty past nseg.
template <int K>
__device__ __forceinline__ void load_slots(const uint2* __restrict__ slots,
                                           const uint32_t* __restrict__ perm, int ss,
                                           uint64_t first, uint64_t nseg, uint2 (&v)[K]) {
  // K divides 2^ss: a thread's slots are one query's, all there or none is.
  if (first < nseg) {
    if (perm) first = ((uint64_t)perm[first >> ss] << ss) + (first & ((1u << ss) - 1));
    if constexpr (K == 1) {
      v[0] = slots[first];
    } else {
#pragma unroll
      for (int i = 0; i < K; i += 2) {
        const uint4 t = ((const uint4*)(slots + first))[i / 2];
        v[i] = make_uint2(t.x, t.y);
        v[i + 1] = make_uint2(t.z, t.w);
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] = make_uint2(0, 0);
  }
}

// Rows of each workgroup's K * 256 slots, from the slots (where the search
// kernel's workgroups do not hold the queries of as many consecutive places).
template <int K>
__global__ __launch_bounds__(256) void slot_rows(const uint2* __restrict__ slots,
                                                 const uint32_t* __restrict__ perm, int ss,
                                                 uint64_t nseg, uint64_t* __restrict__ blk_rows) {
  __shared__ uint64_t s_w[4];
  uint2 v[K];
  load_slots<K>(slots, perm, ss, ((uint64_t)blockIdx.x * 256 + threadIdx.x) * K, nseg, v);
  uint64_t t = 0, total;
#pragma unroll
  for (int i = 0; i < K; ++i) t += rows_of(v[i].y);
  scan256_u64(t, s_w, &total);
  if (threadIdx.x == 0) blk_rows[blockIdx.x] = total;
}

// What a wave's lanes stored to LDS before, its lanes load after.  (The barrier alone
// holds the instructions' order; the fences also keep a lane from taking what it
// stored itself for what is there.)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Whether the batch is left alone, not tested and nothing of it written: it has more
// rows than a capacity (flagged; it is compacted again, or reported), or one of the
// error bits that its caller rejects it for.
__device__ __forceinline__ void put_verdict(BatchStatus* status, uint64_t max_rows64,
                                            uint32_t reject) {
  const bool over = status->rows > max_rows64;
  const uint32_t err = status->err;
  if (over) status->err = err | kErrOverflow;
  status->left = over || (err & reject) != 0 ? 1u : 0u;
}

// Row descriptors of a launch's rows [rbase, rend): for row r of slot s, the
// first sorted index of the row and the query (row_meta) and the number of its
// candidates (row_info), and the first row of every place (row_off).  One block
// per K * 256 slots (whole queries: 2^ss slots each), a thread's K slots
// consecutive; the block's rows are spread over its waves, 64 at a time: the slots
// that start among them mark their first row in LDS, and a row's slot is that of
// the last mark up to it.  FUSED (at most kFusedBlocks blocks): the block sums the
// rows of the blocks before it itself and block 0 gathers the batch's counters, so
// that a small batch takes no batch_scan launch (5 us; with more blocks the
// repeated sums would cost more).
constexpr uint32_t kFusedBlocks = 1024;

template <int K, bool FUSED>
__global__ __launch_bounds__(256) void expand_rows(
    uint64_t* __restrict__ row_off, const uint2* __restrict__ slots,
    const uint32_t* __restrict__ perm, const uint64_t* __restrict__ blk_rows,
    const uint64_t* __restrict__ blk_off, const GroupSums* __restrict__ groups, BatchStats B,
    BatchStatus* status, uint64_t m, int ss, uint64_t rbase, uint64_t row_end, uint64_t max_rows64,
    uint32_t reject, uint2* __restrict__ row_meta, uint16_t* __restrict__ row_info) {
  __shared__ uint64_t st[256 * K + 1];
  __shared__ uint2 s_slot[256 * K];
  __shared__ uint16_t s_mark[4][kWave];
  __shared__ uint32_t s_query[64];   // of the block's places (at most 64)
  __shared__ uint64_t s_w[4];
  const uint64_t nseg = m << ss;
  const uint32_t tid = threadIdx.x;
  uint64_t row0 = 0, total = 0;
  if (FUSED) {
    uint64_t before = 0, all = 0;
    for (uint32_t i = tid; i < gridDim.x; i += 256) {
      const uint64_t v = blk_rows[i];
      all += v;
      before += i < blockIdx.x ? v : 0;
    }
    scan256_u64(before, s_w, &row0);
    scan256_u64(all, s_w, &total);
    if (blockIdx.x == 0) {
      sum_stats<4>(B, status, nullptr);
      if (tid == 0) {
        row_off[m] = total;
        put_verdict(status, max_rows64, reject);
      }
    }
  } else {
    row0 = blk_off[blockIdx.x] + (groups ? groups[blockIdx.x / kGroupBlocks].rows : 0);
    total = row_off[m];
    if (blockIdx.x == 0 && tid == 0) put_verdict(status, max_rows64, reject);
  }
  const uint64_t rend = total < row_end ? total : row_end;
  const uint64_t s0 = (uint64_t)blockIdx.x * 256 * K;
  const uint64_t first = s0 + (uint64_t)tid * K;
  const uint64_t place = (s0 >> ss) + tid;   // s0 is a multiple of 2^ss
  if (tid < ((256u * K) >> ss) && place < m) s_query[tid] = perm ? perm[place] : (uint32_t)place;
  uint2 v[K];
  load_slots<K>(slots, perm, ss, first, nseg, v);
  uint64_t mine = 0, here;
#pragma unroll
  for (int i = 0; i < K; ++i) mine += rows_of(v[i].y);
  uint64_t run = row0 + scan256_u64(mine, s_w, &here);
  if (first < nseg && (first & ((1u << ss) - 1)) == 0) row_off[first >> ss] = run;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    st[tid * K + i] = run;
    s_slot[tid * K + i] = v[i];
    run += rows_of(v[i].y);
  }
  if (tid == 255) st[256 * K] = run;
  __syncthreads();
  const uint64_t r0 = st[0] > rbase ? st[0] : rbase;
  const uint64_t r1 = st[256 * K] < rend ? st[256 * K] : rend;
  if (r1 <= r0) return;
  // Each wave takes a quarter of the rows, 64 at a time (by slots, with fewer
  // steps before the first row, one wave often has most of the rows).
  const uint32_t lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t per = ((r1 - r0 + 255) >> 8) << 6;
  const uint64_t first_row = r0 + wv * per;
  const uint64_t last_row = first_row + per < r1 ? first_row + per : r1;
  if (first_row >= last_row) return;   // the whole wave; no barrier follows
  // The last slot that starts at or before the first row.
  uint32_t k0 = 0;
#pragma unroll
  for (uint32_t i = 0; i < 4 * K; ++i)
    k0 += (uint32_t)__popcll(__ballot(st[i * kWave + lane] <= first_row));
  k0 -= 1;
  uint16_t* mark = s_mark[wv];
  for (uint64_t base = first_row; base < last_row; base += kWave) {
    // The slots that start in these rows leave their number at their first row;
    // a row's slot is that of the last such row up to it, or the first row's.
    mark[lane] = 0xFFFFu;
    wave_sync();
    for (uint32_t k = k0 + 1; k < 256 * K && st[k] < base + kWave; k += kWave) {
      const uint32_t mine = k + lane;
      if (mine < 256 * K && s_slot[mine].y != 0) {
        const uint64_t at = st[mine] - base;   // (a slot before the base wraps)
        if (at < kWave) mark[at] = (uint16_t)mine;
      }
    }
    wave_sync();
    const uint32_t own = mark[lane];
    const uint64_t starts = __ballot(own != 0xFFFFu) & (~0ull >> (63 - lane));
    const uint32_t k = starts ? mark[63 - __clzll(starts)] : k0;
    wave_sync();
    const uint64_t r = base + lane;
    if (r < last_row) {
      const uint64_t local = (r - st[k]) << kRowShift;
      const uint2 sl = s_slot[k];
      const uint64_t left = sl.y - local;
      row_meta[r - rbase] = make_uint2((uint32_t)(sl.x + local),
                                       s_query[k >> ss]);
      row_info[r - rbase] = (uint16_t)(left < 32 ? left : 32);
    }
    k0 = __builtin_amdgcn_readlane(k, 63);
  }
}

// What a query's limits are compared with, from the quanta between its cell and a
// candidate's on each axis: the sum of their squares, or (WINDOW) the largest.
template <int DIM, bool WINDOW>
__device__ __forceinline__ float cell_distance(const int32_t (&off)[3]) {
  float e[DIM];
#pragma unroll
  for (int a = 0; a < DIM; ++a) e[a] = (float)off[a];
  if (WINDOW) {
    float v = fabsf(e[0]);
#pragma unroll
    for (int a = 1; a < DIM; ++a) v = fmaxf(v, fabsf(e[a]));
    return v;
  }
  float v = e[0] * e[0];
#pragma unroll
  for (int a = 1; a < DIM; ++a) v = __fmaf_rn(e[a], e[a], v);
  return v;
}

// The exact test of candidate pos against query qs (the point and the query
// read here: only for candidates their cell could not decide).  The point
// is src[pos] (sorted points), or src[via[pos]] (input order, via = ids).
template <int DIM>
__device__ __forceinline__ bool exact_hit(const double* __restrict__ q,
                                          const double* __restrict__ delta,
                                          const double* __restrict__ src,
                                          const uint32_t* __restrict__ via, uint32_t qs,
                                          uint32_t pos, bool window) {
  const double d = delta[qs];
  const uint64_t at = via ? via[pos] : pos;
  if (DIM == 2) {
    const double2 qq = ((const double2*)q)[qs];
    const double2 p = ((const double2*)src)[at];
    return window ? within_window(p.x, p.y, qq.x, qq.y, d) : within(p.x, p.y, qq.x, qq.y, d);
  }
  const double* qp = q + 3 * (uint64_t)qs;
  const double* pp = src + 3 * at;
  return window ? within_window3(pp[0], pp[1], pp[2], qp[0], qp[1], qp[2], d)
                : within3(pp[0], pp[1], pp[2], qp[0], qp[1], qp[2], d);
}

// A predicate for this lane from a mask that is the same in every lane.
__device__ __forceinline__ bool lane_of(uint64_t mask) {
  return __builtin_amdgcn_inverse_ballot_w64(mask);
}

// Lane R's word replaced by v's low word and lane R + 32's by its high one (v the
// same in every lane).  A vector instruction may read a scalar that another
// wrote (the compares that made v) only two wait states later, which the
// compiler does not see to in inline assembly: hence the s_nop.
template <int R>
__device__ __forceinline__ void write_pair(uint64_t v, uint32_t& w) {
  asm("s_nop 1\n\tv_writelane_b32 %0, %1, %3\n\tv_writelane_b32 %0, %2, %4"
      : "+v"(w)
      : "s"(__builtin_amdgcn_readfirstlane((uint32_t)v)),
        "s"(__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32))), "n"(R), "n"(R + 32));
}

// f(0), f(1), ..., f(N - 1) with the index a constant of its type.
template <typename F, int... I>
__device__ __forceinline__ void static_for_each(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_each(std::make_integer_sequence<int, N>{}, f);
}

// Set bits of a mask below this lane.
__device__ __forceinline__ uint32_t below_in(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// Lane R's word, as a scalar.
template <int R>
__device__ __forceinline__ uint32_t read_lane(uint32_t v) {
  return __builtin_amdgcn_readlane(v, R);
}

// In every row of 16 lanes, the word of its lane T, in a register of its own: the
// compiler would fold the permutation into the instruction using the word, and in
// those of reversed operands (v_subrev, v_lshrrev) the hardware then permutes the
// other operand (measured).  The moves cost the passes nothing that shows: they wait
// for memory (2^20 queries over 2^24 points 2091 and 2094 us a step without and with
// the three that were folded before, 2^22 over 2^26 1547 and 1550).
template <int T>
__device__ __forceinline__ uint32_t bcast16(uint32_t v) {
  return permute_lanes<0x150 + T>(v);
}
template <int T>
__device__ __forceinline__ uint64_t bcast16(uint64_t v) {
  return (uint64_t)bcast16<T>((uint32_t)(v >> 32)) << 32 | bcast16<T>((uint32_t)v);
}
// Every lane's word plus those of the lanes below it in its row of 16.
__device__ __forceinline__ uint32_t scan16(uint32_t v) {
  v += permute_lanes<0x111>(v);   // of the lane 1 below, 0 for none
  v += permute_lanes<0x112>(v);   // 2
  v += permute_lanes<0x114>(v);   // 4
  v += permute_lanes<0x118>(v);   // 8
  return v;
}

// Rows of a wave's unit: step t takes rows 2t (lanes 0..31) and 2t + 1, and
// lane l holds what belongs to row 2 (l % 16) + l / 32 (lanes with bit 4 set
// what those 16 below hold), so that in step t bcast16<t> gives each lane what
// belongs to its row.
__device__ __forceinline__ uint32_t unit_row(uint32_t lane) {
  return 2 * (lane & 15) + (lane >> 5);
}

typedef double f64x2 __attribute__((ext_vector_type(2)));

// Rows of a wave's unit that exist (row0: its first row within the chunk of
// `have` rows).
__device__ __forceinline__ uint32_t unit_rows(uint64_t have, uint64_t row0) {
  return have <= row0 ? 0u : (uint32_t)(have - row0 < kUnitRows ? have - row0 : kUnitRows);
}

// Pass 1: the exact test of every candidate; per row the 32-bit mask of the
// accepted ones (masks) and the number of accepted ones in the unit's rows before
// it (row_info, which held the row's candidates), per unit (a wave's 32 rows) their
// number.  A wave writes its masks, prefixes and count with one store each, so
// that the waves of a workgroup never wait for each other and nothing is cleared
// beforehand.  EPOCH: a candidate that passes the test also has to be visible at
// the query's epoch (ins <= e < era); only those lanes read the epochs.
// window: the square-window test instead of the Euclidean one.
//
// The pass is bound by the vector instructions of a step (two rows) and by the
// latency of its chain of loads (descriptor, record, candidates).  So the lanes
// hold the 32 rows' descriptors and records, loaded for all rows at once and one
// unit ahead, and a step's lanes get their row's words by a broadcast in each row
// of 16 lanes; STEPS steps' candidates are read at a time, a group's loads leaving
// before the previous group is tested; the two verdicts are masks straight from the
// compares.
// Measured (rows of 64, one at a time, before): 0.302 ms for the 4 * 10^8
// candidates of 2 * 10^5 windows in curve order (0.282), the caches' 12 TB/s its
// limit; 0.32 ms for 3.7 * 10^8 of 2^20 queries over 2^24 points (0.365); 0.508
// ms for 2.4 * 10^8 of 2^22 queries in no order, 19 a range (0.677), memory's
// 6.5 TB/s.
template <int STEPS, int ITERS, bool EPOCH, int DIM, bool CELLS, bool WINDOW, bool SHIFTS>
__global__ __launch_bounds__(256) void compact_test(
    const double* __restrict__ q, const double* __restrict__ delta, uint64_t m,
    const double* __restrict__ pts, const uint32_t* __restrict__ via,
    const uint64_t* __restrict__ cells, const void* __restrict__ rec,
    const uint2* __restrict__ row_meta, const uint64_t* __restrict__ total_rows_dev,
    uint64_t rbase, uint64_t row_end, uint32_t* __restrict__ masks,
    uint16_t* __restrict__ row_info, uint32_t* __restrict__ unit_hits, BatchStatus* status,
    const uint32_t* __restrict__ ins, const uint32_t* __restrict__ era) {
  static_assert(STEPS * ITERS == kUnitSteps, "a wave's groups cover its rows");
  static_assert(!(EPOCH && CELLS), "an index with epochs keeps no cells");
  const uint32_t lane = lane_id(), row = unit_row(lane), lane32 = lane & 31;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // SHIFTS: the batch may hold queries with coarser cells
  const bool any_shifted = SHIFTS && CELLS && status->coarse != 0u;
  const uint64_t total_all = *total_rows_dev;
  const uint64_t total_rows = total_all < row_end ? total_all : row_end;
  const uint64_t ntiles = chunk_tiles(total_all, rbase, row_end, status->left != 0);
  const uint64_t have = total_rows - rbase;
  // What belongs to a lane's row: its descriptor (rows past the last: candidate 0
  // of query 0, whose result is dropped), then the record of its query.  A
  // record is four or eight words; the plane's cell filter needs the first four,
  // and its shift (the sixth) only in a batch with coarser cells.
  constexpr int kRecWords = CELLS && DIM == 2 && !SHIFTS ? 4 : 8;
  // (Loaded words are kept as they come: arithmetic on them here would wait for
  // them here.)
  struct Unit {
    uint32_t pb, nv, at;
    uint32_t rec[kRecWords];
  };
  auto fetch_rows = [&](uint64_t tile, Unit& u) {
    u.pb = u.at = 0;
    u.nv = 1;
    const uint64_t row0 = tile * kTileRows + (uint64_t)w * kUnitRows;
    if (tile != ~0ull && row < unit_rows(have, row0)) {
      const uint2 md = row_meta[row0 + row];
      u.pb = md.x;
      u.at = md.y;
      u.nv = row_info[row0 + row];
    }
  };
  auto fetch_rec = [&](Unit& u) {
    const uint4* r = (const uint4*)rec + 2 * (uint64_t)u.at;
#pragma unroll
    for (int i = 0; i < kRecWords; i += 4) {
      const uint4 v = r[i / 4];
      u.rec[i] = v.x;
      u.rec[i + 1] = v.y;
      u.rec[i + 2] = v.z;
      u.rec[i + 3] = v.w;
    }
  };
  uint64_t tile = xcd_tile(blockIdx.x, gridDim.x, 0, ntiles);
  if (tile != ~0ull) {
    Unit u, nx;
    fetch_rows(tile, u);
    fetch_rec(u);
    uint64_t next = xcd_tile(blockIdx.x, gridDim.x, 1, ntiles);
    fetch_rows(next, nx);
    for (uint64_t step = 2;; ++step) {
      const uint64_t row0 = tile * kTileRows + (uint64_t)w * kUnitRows;
      const uint64_t after = next == ~0ull ? ~0ull
                                           : xcd_tile(blockIdx.x, gridDim.x, step, ntiles);
      Unit nn;
      fetch_rows(after, nn);
      fetch_rec(nx);   // the next unit's records, its descriptors being here
      // The last of the row's lanes that has a candidate (the lanes past it
      // repeat its candidate, and their verdicts are dropped at the end).
      const uint32_t ulast = u.nv - 1;
      uint32_t mk = 0;   // the mask of the lane's row (lanes without bit 4)

      // The sorted index of the lane's candidate in step t.
      auto position = [&](auto t) {
        constexpr int T = decltype(t)::value;
        const uint32_t last = bcast16<T>(ulast);
        return bcast16<T>(u.pb) + (lane32 < last ? lane32 : last);
      };
      // A group's candidates: one load per step (three coordinates: three).
      struct Group {
        uint64_t cell[CELLS ? STEPS : 1];
        f64x2 xy[CELLS ? 1 : STEPS];
        double z[CELLS || DIM == 2 ? 1 : STEPS];
      };
      auto load = [&](auto group, Group& G) {
        static_for<STEPS>([&](auto i) {
          constexpr int g = decltype(i)::value, t = decltype(group)::value * STEPS + g;
          const uint64_t pos = position(std::integral_constant<int, t>{});
          if constexpr (CELLS) {
            G.cell[g] = cells[pos];
          } else if constexpr (DIM == 2) {
            G.xy[g] = ((const f64x2*)pts)[pos];
          } else {
            G.xy[g].x = pts[3 * pos];
            G.xy[g].y = pts[3 * pos + 1];
            G.z[g] = pts[3 * pos + 2];
          }
        });
      };
      auto test = [&](auto group, const Group& G, auto shifted) {
        uint64_t hit[STEPS], und[STEPS], any = 0;
        static_for<STEPS>([&](auto i) {
          constexpr int g = decltype(i)::value, t = decltype(group)::value * STEPS + g;
          if constexpr (CELLS) {
            // Decide from the cells.
            // (A shifted query's cells are compared 2^shift quanta wide.)
            const float acc = __uint_as_float(bcast16<t>(u.rec[0]));
            const float rej = __uint_as_float(bcast16<t>(u.rec[1]));
            constexpr bool kShifted = decltype(shifted)::value;
            const uint32_t shift = kShifted ? bcast16<t>(u.rec[kRecWords > 4 ? 5 : 0]) : 0u;
            constexpr int B = DIM == 2 ? 32 : 21;
            auto axis = [&](auto k) {
              constexpr int a = decltype(k)::value;
              uint32_t c = (uint32_t)((G.cell[g] >> (B * a)) & ((1ull << B) - 1));
              if (kShifted) c >>= shift;
              return (int32_t)(c + bcast16<t>(u.rec[kRecWords > 4 || a < 2 ? 2 + a : 0]));
            };
            int32_t off[3] = {axis(std::integral_constant<int, 0>{}),
                              axis(std::integral_constant<int, 1>{}), 0};
            if constexpr (DIM == 3) off[2] = axis(std::integral_constant<int, 2>{});
            const float v = cell_distance<DIM, WINDOW>(off);
            const uint64_t in = __ballot(v <= acc), out = __ballot(v > rej);
            hit[g] = in;
            und[g] = ~(in | out);
            any |= und[g];
          } else {
            auto word = [&](auto k) {
              constexpr int c = decltype(k)::value;
              return __longlong_as_double((long long)((uint64_t)bcast16<t>(u.rec[c + 1]) << 32 |
                                                      bcast16<t>(u.rec[c])));
            };
            const double qx = word(std::integral_constant<int, 0>{});
            const double qy = word(std::integral_constant<int, 2>{});
            const double third = word(std::integral_constant<int, 4>{});
            bool h;
            if constexpr (DIM == 2) {
              h = WINDOW ? within_window(G.xy[g].x, G.xy[g].y, qx, qy, third)
                         : within(G.xy[g].x, G.xy[g].y, qx, qy, third);
            } else {
              const double d = word(std::integral_constant<int, 6>{});
              h = WINDOW ? within_window3(G.xy[g].x, G.xy[g].y, G.z[g], qx, qy, third, d)
                         : within3(G.xy[g].x, G.xy[g].y, G.z[g], qx, qy, third, d);
            }
            hit[g] = __ballot(h);
          }
        });
        if constexpr (CELLS) {
          // The candidates their cells leave undecided (rare) take the exact
          // test, behind one branch for the whole group.
          if (any != 0)
            static_for<STEPS>([&](auto i) {
              constexpr int g = decltype(i)::value, t = decltype(group)::value * STEPS + g;
              const uint32_t pos = position(std::integral_constant<int, t>{});
              const uint32_t at = bcast16<t>(u.at);
              bool h = false;
              if (lane_of(und[g])) h = exact_hit<DIM>(q, delta, pts, via, at, pos, WINDOW);
              hit[g] |= __ballot(h);
            });
        }
        if constexpr (EPOCH)
          static_for<STEPS>([&](auto i) {
            constexpr int g = decltype(i)::value, t = decltype(group)::value * STEPS + g;
            const uint32_t pos = position(std::integral_constant<int, t>{});
            const uint32_t qe = bcast16<t>(u.rec[kRecWords > 4 ? 7 : 0]);
            bool h = false;
            if (lane_of(hit[g])) h = ins[pos] <= qe && qe < era[pos];
            hit[g] = __ballot(h);
          });
        static_for<STEPS>([&](auto i) {
          constexpr int g = decltype(i)::value, t = decltype(group)::value * STEPS + g;
          write_pair<t>(hit[g], mk);
        });
      };
      auto groups = [&](auto shifted) {
        Group G[2];
        load(std::integral_constant<int, 0>{}, G[0]);
        static_for<ITERS>([&](auto group) {
          constexpr int g = decltype(group)::value;
          if constexpr (g + 1 < ITERS) load(std::integral_constant<int, g + 1>{}, G[(g + 1) & 1]);
          // (Every load of the group first: else a wait for one comes before the next.)
          __builtin_amdgcn_sched_barrier(0);
          test(group, G[g & 1], shifted);
          __builtin_amdgcn_sched_barrier(0);
        });
      };
      // A batch with coarser cells (radii past the shift limit) takes the shifting
      // check throughout (one branch per unit: with one per step the steps' loads
      // and compares did not overlap).
      if (SHIFTS && CELLS && any_shifted) groups(std::integral_constant<bool, SHIFTS && CELLS>{});
      else groups(std::integral_constant<bool, false>{});

      // The rows' valid hits, and the unit's before the row: those of the pairs
      // of rows before, and of the pair's first row before its second.
      const uint32_t mask = row < unit_rows(have, row0) ? mk & (~0u >> (31 - ulast)) : 0;
      const uint32_t v = __popc(mask), other = __shfl_xor(v, 32, 64);
      const uint32_t upto = scan16(v + other);
      if ((lane & 16) == 0) {
        masks[row0 + row] = mask;
        row_info[row0 + row] = (uint16_t)(upto - (lane < 32 ? v + other : v));
        if (lane == 15) unit_hits[tile * kTileUnits + w] = upto;
      }
      if (next == ~0ull) break;
      u = nx;
      nx = nn;
      tile = next;
      next = after;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) status->units = (uint32_t)(ntiles * kTileUnits);
}

// Hits before the unit: of every unit (of `units`), and at [units] all hits,
// in LDS, from the units' hits (FUSED compaction: at most kFusedUnits).
constexpr uint32_t kFusedUnits = 4096;

__device__ __forceinline__ void units_to_lds(const uint32_t* __restrict__ unit_hits,
                                             uint32_t units, uint32_t* s_off, uint64_t* s_w) {
  constexpr uint32_t kPer = kFusedUnits / 256;
  const uint32_t f = threadIdx.x * kPer;
  uint32_t v[kPer], sum = 0;
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) v[i] = f + i < units ? unit_hits[f + i] : 0u;
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) sum += v[i];
  uint64_t total;
  uint32_t run = (uint32_t)scan256_u64(sum, s_w, &total);
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    s_off[f + i] = run;
    run += v[i];
  }
  if (threadIdx.x == 255) s_off[kFusedUnits] = run;
  __syncthreads();
}

// Pass 2: the ids of the accepted candidates.  A wave takes a unit of 32 rows, two
// at a time as in the test pass: the lanes of a row's mask read their ids and write
// them one after another from the row's place in the output.  ORDERED (rows in
// curve order): that is the query's output offset plus the query's hits before
// the row, out_base[query] + P(row) with P(row) the hits of all rows before it;
// else rows follow the output, P(row) is the place, and the workgroups past
// `tile_grid` write the queries' CSR offsets, P of each query's first row.
// FUSED (at most kFusedUnits units): every workgroup scans the units' hits
// itself, so that a small batch takes no scan launch.  The batch's final
// counters go to *host (host memory) and its error bits to *flags_out, if not
// null.  Bound by memory: 0.362 ms for 0.81 GB of ids of 4 * 10^8 candidates, 3.5
// TB/s with what is read (0.378 for rows of 64, 0.43 with a workgroup's hits
// listed in LDS first; 0.245 ms, 0.313 for rows of 64, for 0.17 GB of 2.4 * 10^8).
// Listing a wave's hits in LDS, for loads and stores of 64 lanes, takes a third of
// the memory instructions but a tenth more time; non-temporal stores are better
// (0.355) only where a query reports a thousand ids (0.41 for 0.36 at 170).
template <bool ORDERED, bool FUSED>
__global__ __launch_bounds__(256) void compact_write_out(
    const uint32_t* __restrict__ ids, const uint2* __restrict__ row_meta,
    const uint64_t* __restrict__ row_off, uint64_t m, uint64_t rbase, uint64_t rend,
    uint64_t row_end, const uint32_t* __restrict__ masks,
    const uint16_t* __restrict__ row_info, const uint32_t* __restrict__ unit_hits,
    const uint64_t* __restrict__ unit_off, const uint64_t* __restrict__ out_base,
    uint32_t tile_grid, uint32_t* __restrict__ out_ids,
    uint64_t cap, bool whole, uint64_t* __restrict__ offsets, const BatchStatus* status,
    BatchStatus* host, uint32_t* flags_out) {
  __shared__ uint32_t s_off[FUSED ? kFusedUnits + 1 : 1];
  __shared__ uint64_t s_w[4];
  static_assert(!(ORDERED && FUSED), "small batches are not ordered");
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint64_t total_all = row_off[m];
  const uint64_t total_rows = total_all < row_end ? total_all : row_end;
  const bool over = status->left != 0;
  const uint64_t ntiles = chunk_tiles(total_all, rbase, row_end, over);
  const uint64_t units = ntiles * kTileUnits;
  // A workgroup without a tile (and not the first, which reports) is done.
  if (blockIdx.x > 0 && blockIdx.x < tile_grid &&
      xcd_tile(blockIdx.x, tile_grid, 0, ntiles) == ~0ull)
    return;
  if (FUSED) units_to_lds(unit_hits, (uint32_t)units, s_off, s_w);
  // All hits up to the end of this chunk; without rows in it there are none
  // to write (and, in the first chunk, none at all).
  const uint64_t hits_end = FUSED ? s_off[units] : ntiles ? unit_off[units] : 0;
  // The chunk owns rows [rbase, rend) below the total and, if the total falls
  // in (rbase, rend], the total itself.
  const bool owns_total = total_rows == 0 ? rbase == 0 : (rbase < total_rows && total_rows <= rend);
  if (blockIdx.x == 0 && tid == 0) {
    if (host && owns_total) {
      host->rows = status->rows;
      host->total = ORDERED ? offsets[m] : hits_end;
      host->candidates = status->candidates;
      host->endpoints = status->endpoints;
      host->fallbacks = status->fallbacks;
      host->pruned = status->pruned;
      host->err = status->err;
      host->coarse = status->coarse;
    }
    if (flags_out) *flags_out = status->err;
  }
  if (over) return;   // nothing was tested
  if (!ORDERED && blockIdx.x >= tile_grid) {
    // The CSR offsets of the queries whose first row lies in this chunk (a
    // query with no rows takes the position of the next row, trailing ones
    // the total).
    const uint64_t stride = (uint64_t)(gridDim.x - tile_grid) * 256;
    for (uint64_t j = (uint64_t)(blockIdx.x - tile_grid) * 256 + tid; j <= m; j += stride) {
      uint64_t r = row_off[j];
      if (r > total_rows) r = total_rows;   // past the capacity (flagged as overflow)
      if (r == total_rows) {
        if (owns_total) offsets[j] = hits_end;
      } else if (r >= rbase && r < rend) {
        const uint64_t lr = r - rbase;
        offsets[j] = (FUSED ? (uint64_t)s_off[lr >> kUnitShift] : unit_off[lr >> kUnitShift]) +
                     row_info[lr];
      }
    }
    return;
  }
  const bool write_ids = !whole || ntiles == 0 || (ORDERED ? offsets[m] : hits_end) <= cap;
  if (!write_ids) return;
  const uint64_t have = total_rows - rbase;
  // What belongs to a lane's row: its mask and first position, and the terms of
  // its place in the output (kept as they come, not to wait for them here).
  const uint32_t row = unit_row(lane), lane32 = lane & 31;
  struct Unit {
    uint64_t unit, base;
    uint32_t mask, pb, at;
  };
  auto fetch_rows = [&](uint64_t tile, Unit& u) {
    u.unit = u.base = 0;
    u.mask = u.pb = u.at = 0;
    const uint64_t row0 = tile * kTileRows + (uint64_t)w * kUnitRows;
    if (tile != ~0ull && row < unit_rows(have, row0)) {
      const uint64_t lr = row0 + row;
      u.mask = masks[lr];
      const uint2 md = row_meta[lr];
      u.pb = md.x;
      u.at = md.y;
      u.unit = FUSED ? (uint64_t)s_off[lr >> kUnitShift] : unit_off[lr >> kUnitShift];
    }
  };
  auto fetch_base = [&](Unit& u) {
    if (ORDERED) u.base = out_base[u.at];
  };
  uint64_t tile = xcd_tile(blockIdx.x, tile_grid, 0, ntiles);
  if (tile == ~0ull) return;
  Unit u, nx;
  fetch_rows(tile, u);
  fetch_base(u);
  uint64_t next = xcd_tile(blockIdx.x, tile_grid, 1, ntiles);
  fetch_rows(next, nx);
  for (uint64_t step = 2;; ++step) {
    const uint64_t after = next == ~0ull ? ~0ull : xcd_tile(blockIdx.x, tile_grid, step, ntiles);
    Unit nn;
    fetch_rows(after, nn);
    fetch_base(nx);
    // The row's place; the capacity checked once for the unit.
    const uint32_t v = __popc(u.mask), other = __shfl_xor(v, 32, 64);
    const uint32_t upto = scan16(v + other);
    const uint64_t place = u.unit + u.base + (upto - (lane < 32 ? v + other : v));
    const bool fits = __ballot(place + 32 > cap) == 0;
    // A step's hits are counted over both rows: the second row's start counts
    // the first one's hits off.
    const uint64_t to = place - (lane < 32 ? 0 : other);
    // Lanes past a row's last hit read that one again, and a row without hits the
    // index's first id, which is at hand (not a line of its own).  All the ids are waited
    // for at once: a wait for one of them after a store would wait for stores
    // too (they share a counter).
    const uint32_t end = u.mask ? 31 - (uint32_t)__clz(u.mask) : 0u;
    const uint32_t pb = u.mask ? u.pb : 0u;
    uint32_t id[kUnitSteps];
    static_for<kUnitSteps>([&](auto t) {
      constexpr int T = decltype(t)::value;
      const uint32_t last = bcast16<T>(end);
      id[T] = ids[(uint64_t)(bcast16<T>(pb) + (lane32 < last ? lane32 : last))];
    });
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    static_for<kUnitSteps>([&](auto t) {
      constexpr int T = decltype(t)::value;
      const uint64_t mk = (uint64_t)read_lane<T + 32>(u.mask) << 32 | read_lane<T>(u.mask);
      const uint64_t at = bcast16<T>(to) + below_in(mk);
      if (lane_of(mk) && (fits || at < cap)) out_ids[at] = id[T];
    });
    if (next == ~0ull) break;
    u = nx;
    nx = nn;
    next = after;
  }
}

// Ordered rows: the hits of every query, and in out_base the hits P of all
// rows before its first.  One thread per place.
__global__ __launch_bounds__(256) void query_hits(const uint64_t* __restrict__ row_off, uint64_t m,
                                                  const BatchStatus* status,
                                                  const uint16_t* __restrict__ row_info,
                                                  const uint64_t* __restrict__ unit_off,
                                                  const uint32_t* __restrict__ perm,
                                                  uint32_t* __restrict__ qhits,
                                                  uint64_t* __restrict__ out_base) {
  const uint64_t at = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (at >= m) return;
  const uint64_t total_all = row_off[m];
  const uint64_t total = status->left ? 0 : total_all;
  const uint64_t units = (total + kTileRows - 1) / kTileRows * kTileUnits;
  auto before = [&](uint64_t r) -> uint64_t {
    if (r >= total) return total ? unit_off[units] : 0;
    return unit_off[r >> kUnitShift] + row_info[r];
  };
  const uint64_t p0 = before(row_off[at]), p1 = before(row_off[at + 1]);
  const uint32_t j = perm[at];
  qhits[j] = (uint32_t)(p1 - p0);
  out_base[j] = p0;
}

// out_base: from P of the query's first row to what added to P(row) gives the
// row's place in the output.
__global__ __launch_bounds__(256) void place_rows(const uint64_t* __restrict__ offsets, uint64_t m,
                                                  uint64_t* __restrict__ out_base) {
  const uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (j < m) out_base[j] = offsets[j] - out_base[j];
}

__global__ void fill64_kernel(uint64_t* p, uint64_t v, uint64_t count) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
    p[i] = v;
}
__global__ void fill32_kernel(uint32_t* p, uint32_t v, uint64_t count) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
    p[i] = v;
}

// Tiles per compaction chunk (lowered only by the test hook).
std::atomic<uint64_t> g_chunk_tiles{kCompactChunkTiles};

// Shape of the test kernel's groups, steps x iterations: 0: 16 x 1, 1: 4 x 4,
// 2: 8 x 2, 3: 2 x 8, 4: 1 x 16 (same results for all).  The environment
// variable SFC_TEST_VARIANT overrides; else the autotuner's choice for this number
// of rows; else 1 (2^20 queries over 2^24 points: 0.322 ms, 0.322 for 16 x 1,
// 0.321 for 8 x 2 and 0.331 for 2 x 8).
int test_variant(uint64_t rows) {
  static const int env = [] {
    const char* e = std::getenv("SFC_TEST_VARIANT");
    return e ? std::atoi(e) + 1 : 0;
  }();
  const int v = env ? env - 1 : tuned(kTuneTestShape, rows);
  return v >= 0 && v <= 4 ? v : 1;
}

uint32_t fill_blocks(uint64_t count) {
  uint64_t b = (count + 255) / 256;
  if (b > 2048) b = 2048;
  return b < 1 ? 1 : (uint32_t)b;
}

}  // namespace

uint64_t compact_chunk_tiles() { return g_chunk_tiles.load(std::memory_order_relaxed); }
bool compact_single_chunk(uint64_t total_rows) {
  return (total_rows + kCompactTileRows - 1) / kCompactTileRows <= compact_chunk_tiles();
}
void set_compact_chunk_tiles(uint64_t tiles) {
  g_chunk_tiles.store(tiles == 0 || tiles > kCompactChunkTiles ? kCompactChunkTiles : tiles,
                      std::memory_order_relaxed);
}

hipError_t fill_u64(uint64_t* p, uint64_t value, uint64_t count, hipStream_t s) {
  if (count == 0) return hipSuccess;
  fill64_kernel<<<fill_blocks(count), 256, 0, s>>>(p, value, count);
  return hipGetLastError();
}
hipError_t fill_u32(uint32_t* p, uint32_t value, uint64_t count, hipStream_t s) {
  if (count == 0) return hipSuccess;
  fill32_kernel<<<fill_blocks(count), 256, 0, s>>>(p, value, count);
  return hipGetLastError();
}

// The sizes callers plan with (sfc_query_scratch_size, the fixed scratch of
// sfc_query_batch_static): they stay as published, and the layouts below use
// less (checked where they are carved).
size_t query_scratch_bytes(uint64_t m, uint32_t slots) {
  const uint64_t nseg = slots * m;
  return align256(nseg * 4) * 3 + align256((nseg + 1) * 8) + scan_scratch_bytes(nseg) +
         align256(64) + align256(4 * m * 8) + align256(m * 32) + align256(m * 4) +
         order_scratch_bytes(m) + align256(m * 4);
}

bool query_scratch_carve(void* base, uint64_t m, QueryScratch* qs, uint32_t slots) {
  const uint64_t nseg = slots * m;
  const uint64_t nblk = (m + 31) / 32;           // search workgroups (32 or 64 queries each)
  const uint64_t npack = (m + 255) / 256;        // cells_pack workgroups
  char* p = (char*)base;
  qs->m = m;
  qs->status = (BatchStatus*)p;   p += align256(sizeof(BatchStatus));
  qs->slots = (uint2*)p;          p += align256(nseg * 8);
  qs->row_off = (uint64_t*)p;     p += align256((m + 1) * 8);
  qs->blk_rows = (uint64_t*)p;
  qs->blk_off = qs->blk_rows + nblk;
  qs->blk_stat = qs->blk_off + nblk;
  qs->blk_rows64 = qs->blk_stat + nblk;
  qs->blk_place = qs->blk_rows64 + nblk;
  qs->blk_learned = (uint32_t*)(qs->blk_place + nblk);
  p += align256(nblk * 44);
  qs->groups = p;
  p += align256((nblk + kGroupBlocks - 1) / kGroupBlocks * sizeof(GroupSums));
  qs->rec = p;                    p += align256(m * 32);
  qs->perm = (uint32_t*)p;        p += align256(m * 4);
  qs->out_base = (uint64_t*)p;    p += align256(m * 8);
  qs->qhits = (uint32_t*)p;       p += align256(m * 4);
  qs->scan_tmp = (uint64_t*)p;    p += scan_scratch_bytes(m);
  // One region for what is needed in turn: the ordering's buffers and the work
  // list of early termination.
  char* aux = p;
  qs->order_scratch = aux;
  const size_t order_end = order_scratch_bytes(m);
  char* e = aux;
  qs->pairs = (uint64_t*)e;       e += align256(4 * m * 8);
  qs->regions = (uint64_t*)e;     e += align256(4 * m * 8);
  qs->pack_flags = (uint64_t*)e;
  qs->pack_cnt = (uint32_t*)(qs->pack_flags + npack);
  qs->pack_pruned = qs->pack_cnt + npack;
  qs->pack_pre = qs->pack_pruned + npack;
  qs->pack_wanted = qs->pack_pre + npack + 1;
  e += align256(npack * 20 + 8);
  p += (size_t)(e - aux) > order_end ? (size_t)(e - aux) : order_end;
  qs->ss = 2;
  qs->perm_made = false;
  qs->fused = false;
  qs->stats_ns = qs->stats_np = 0;
  qs->learned = false;
  return (size_t)(p - (char*)base) <= query_scratch_bytes(m, slots);
}

size_t compact_scratch_bytes(uint64_t total_rows) {
  uint64_t tiles = (total_rows + kCompactTileRows - 1) / kCompactTileRows;
  if (tiles > kCompactChunkTiles) tiles = kCompactChunkTiles;
  if (tiles == 0) tiles = 1;
  const uint64_t rows = tiles * kCompactTileRows;
  return align256(rows * 8) + align256(tiles * 4) + 2 * align256((tiles + 1) * 8) +
         align256(rows * 16) + align256((rows + 1) * 8) + scan_scratch_bytes(tiles);
}

namespace {

struct CompactScratch {
  uint32_t* masks;       // per row
  uint2* meta;           // per row
  uint16_t* info;        // per row
  uint32_t* unit_hits;   // per unit
  uint64_t* unit_off[2]; // per unit, and the total; two, for the chunks in turn
  uint64_t* scan_tmp;
};

// Lays out the scratch of a chunk of `tiles` tiles; false if it needs more
// than compact_scratch_bytes gives.
bool compact_carve(void* base, uint64_t tiles, CompactScratch* c) {
  char* p = (char*)base;
  const uint64_t units = tiles * kTileUnits;
  c->meta = (uint2*)p;           p += align256(tiles * kTileRows * 8);
  c->masks = (uint32_t*)p;       p += align256(tiles * kTileRows * 4);
  c->info = (uint16_t*)p;        p += align256(tiles * kTileRows * 2);
  c->unit_hits = (uint32_t*)p;   p += align256(units * 4);
  c->unit_off[0] = (uint64_t*)p; p += align256((units + 1) * 8);
  c->unit_off[1] = (uint64_t*)p; p += align256((units + 1) * 8);
  c->scan_tmp = (uint64_t*)p;    p += scan_dev_scratch_bytes(units);
  return (size_t)(p - (char*)base) <= compact_scratch_bytes(tiles * kCompactTileRows);
}

// Query slots per thread of the kernels over slots: a workgroup holds the
// queries of one workgroup of the search (64, or 32 in three dimensions).
int slots_per_thread(const QueryScratch& qs) { return (qs.block_queries << qs.ss) / 256; }

uint32_t query_blocks(const QueryScratch& qs) {
  return (uint32_t)((qs.m + qs.block_queries - 1) / qs.block_queries);
}

BatchStats stats_of(const QueryScratch& qs) {
  return BatchStats{qs.blk_stat, qs.blk_rows64, qs.learned ? qs.blk_learned : nullptr, qs.stats_ns,
                    qs.pack_flags, qs.pack_pruned, qs.stats_np};
}

hipError_t launch_slot_rows(const QueryScratch& qs, const uint32_t* perm, uint64_t* blk_rows,
                            hipStream_t s) {
  const uint64_t nseg = qs.m << qs.ss;
  const uint32_t g = query_blocks(qs);
  switch (slots_per_thread(qs)) {
    case 1: slot_rows<1><<<g, 256, 0, s>>>(qs.slots, perm, qs.ss, nseg, blk_rows); break;
    case 2: slot_rows<2><<<g, 256, 0, s>>>(qs.slots, perm, qs.ss, nseg, blk_rows); break;
    default: slot_rows<4><<<g, 256, 0, s>>>(qs.slots, perm, qs.ss, nseg, blk_rows); break;
  }
  return hipGetLastError();
}

// The groups of a batch whose rows are scanned by groups, or null.
GroupSums* scan_groups(const QueryScratch& qs) {
  return query_blocks(qs) > kOneScan ? (GroupSums*)qs.groups : nullptr;
}

// The scan of the workgroups' rows (blk_off within their groups), and with stats
// the batch's counters.
hipError_t launch_rows_scan(const QueryScratch& qs, const uint64_t* blk_rows, bool stats,
                            BatchStatus* host, hipStream_t s) {
  ProfScope ps("scan", s);
  const uint32_t nblk = query_blocks(qs);
  if (GroupSums* groups = scan_groups(qs)) {
    const uint32_t count = (nblk + kGroupBlocks - 1) / kGroupBlocks;
    group_sums<<<count, 256, 0, s>>>(blk_rows, nblk, qs.blk_off, stats_of(qs), stats, groups);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    group_scan<<<1, 256, 0, s>>>(groups, count, qs.row_off + qs.m, stats, qs.status, host);
    return hipGetLastError();
  }
  batch_scan<<<1, 1024, 0, s>>>(blk_rows, nblk, qs.blk_off, qs.row_off + qs.m, stats_of(qs), stats,
                                qs.status, host);
  return hipGetLastError();
}

// After the search: the rows' scan over the search's workgroups and the
// batch's counters, unless expand_rows does both (fused).
hipError_t finish_ranges(QueryScratch& qs, bool need_rows, BatchStatus* host, hipStream_t s) {
  const uint32_t nblk = query_blocks(qs);
  qs.fused = !need_rows && nblk <= kFusedBlocks && qs.stats_np == 0 && !qs.perm_made;
  if (qs.fused) return hipSuccess;
  return launch_rows_scan(qs, qs.perm_made ? qs.blk_place : qs.blk_rows, true, host, s);
}

}  // namespace

// Whether a batch's search takes its queries in curve order: where the order (23 us
// for 2 * 10^5 queries, 33 for 10^6) costs less than the lines it saves, as the
// probes of a workgroup then meet in the same ones.
//   Binary search: 2^20 queries over 2^24 points 0.76 ms against 0.88 (c 1 to 100;
// 10^3: 1.39 against 1.79), 2^18 0.29 against 0.30 (0.46 against 0.53), 2^17 0.188
// against 0.182 (0.288 against 0.299), 2^17 over 2^20 0.160 against 0.147.
//   The learned index and the search tree probe less: only with refined ranges, whose
// crowded cells take more searches, and many candidates a query.  How many is known
// from the handle's last batch alone.  2^20 queries over 2^24 points, ordered against
// not: search tree 1.47 ms against 1.95 with 360 candidates a query, 0.66 against 0.65
// with 100, 0.25 against 0.21 with hardly any; learned index 1.39 against 1.63, 0.67
// against 0.72, 0.25 against 0.20; 2^18 queries of 360 0.51 against 0.57 and 0.48 against
// 0.49; not refined 1.80 against 1.82 (360), 0.64 against 0.58 (100).  A handle's first
// batch through the search tree is ordered from 2^20 queries on.
//   Batches of point sets are grouped by set as a rule; early termination has its own
// rule (below).
constexpr uint64_t kOrderMin = (1u << 17) + 1;
constexpr uint64_t kOrderPoints = 1u << 20;
constexpr uint64_t kOrderFirst = 1u << 20;
constexpr double kOrderCandidates = 128.0;
bool search_ordered(const RangePlan& P, bool binary, bool stree, uint64_t m) {
  if (P.occ || P.qset || m < kOrderMin || P.n < kOrderPoints) return false;
  if (binary) return true;
  if (!P.refine || P.dim != 2) return false;
  return P.last_candidates < 0.0 ? stree && m >= kOrderFirst
                                 : P.last_candidates >= kOrderCandidates;
}

// With early termination the queries' cells are listed in curve order if the handle's
// last batch had many candidates, and in its first batch if a sample of 1024 queries
// has at least as many cells that hold points (then known on the device alone, which
// orders the queries or not): 2^20 refined queries over 2^24 points where the points
// are, 360 candidates each, 1.57 ms against 2.84, 100 each 0.77 against 0.92, 40 each
// 0.58 against 0.64; 2^18 of them 0.53 against 0.77 and 0.30 against 0.33.  Among cells
// that are mostly empty the search is short: 0.25 ms against 0.22.  (10^6 windows over
// 10^7 points, mostly empty: the first batch takes 0.27 ms, 0.25 without the sample and
// the order's launches, which do nothing then; the sample inside order_count, by every
// workgroup, takes as long.)
constexpr double kListedCandidates = 16.0;
constexpr uint32_t kListedCells = 1024;

// Whether a batch's rows are processed in curve order: the test pass gains a
// third (0.46 -> 0.30 ms for the 4 * 10^8 candidates of 2 * 10^5 windows), but
// the queries' offsets then take a scan of their hits (0.03 ms; 2^20 queries 0.07
// and 2^22 0.2 ms), and the order 0.03 ms unless the search has made it.  So only
// with many rows of 64 a query: at 33 the windows' batch takes 0.91 ms against
// 1.01; at 8 and with the order made (2^20 queries over 2^24 points) 2.13 against
// 2.19; 2^20 queries over 2^24 points in space (search tree) 3.44 against 3.33.
constexpr uint64_t kOrderRows = 16, kOrderRowsMade = 6;
bool rows_ordered(const CompactPlan& P, const QueryScratch& qs) {
  return P.keys && qs.m >= kOrderMin && P.n >= kOrderPoints &&
         P.max_rows > (qs.perm_made ? kOrderRowsMade : kOrderRows) * qs.m;
}

hipError_t launch_ranges(const RangePlan& P, QueryScratch& qs, hipStream_t s) {
  const uint64_t m = qs.m;
  if (m == 0) return hipSuccess;
  const bool dbg = P.dbg_lo != nullptr;
  const bool refine = P.refine && !dbg;   // the inspected ranges are the method's merged ranges
  const bool d3 = P.dim == 3;
  hipError_t e;
  qs.ss = d3 ? (refine ? 5 : 3) : (refine ? 3 : 2);
  qs.block_queries = d3 ? 32 : 64;
  qs.stats_ns = query_blocks(qs);
  qs.stats_np = 0;
  const bool learned = P.lview != nullptr && P.qset == nullptr;
  const bool stree = !learned && P.sview != nullptr && P.qset == nullptr;
  qs.learned = learned;
  const LearnedView lv = learned ? *P.lview : LearnedView{};
  const StreeView sv = stree ? *P.sview : StreeView{};
  RecordPlan rec = P.record;
  rec.rec = qs.rec;
  if (dbg) rec = RecordPlan{};
  const uint32_t* perm = nullptr;
  qs.perm_made = !dbg && search_ordered(P, !learned && !stree, stree, m);
  if (qs.perm_made) {
    if ((e = order_queries(P.q, m, d3 ? SFC_CURVE_MORTON3 : P.curve, P.keys, P.n, qs.perm,
                           qs.order_scratch, s)) != hipSuccess)
      return e;
    perm = qs.perm;
  }
  uint64_t* blk_rows = perm ? qs.blk_place : qs.blk_rows;
  if (d3) {
    ProfScope ps(stree ? "ranges_stree3" : "ranges_search3", s);
#define SFC_R3(S, R)                                                                         \
  ranges_search3<S, R><<<query_blocks(qs), 256, 0, s>>>(P.q, P.delta, m, P.keys, P.n, lv, sv, \
                                                        P.refine_min, perm, rec, qs.slots,   \
                                                        blk_rows, qs.blk_stat,               \
                                                        qs.blk_rows64)
    if (stree) {
      if (refine) SFC_R3(2, true);
      else SFC_R3(2, false);
    } else {
      if (refine) SFC_R3(0, true);
      else SFC_R3(0, false);
    }
#undef SFC_R3
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return finish_ranges(qs, P.need_rows, P.host, s);
  }
  // With early termination (and no inspected ranges) the search runs one
  // lane per surviving cell, from a dense list of (query, cell) pairs.
  const bool dense = P.occ != nullptr && !dbg;
  const uint64_t* pairs = nullptr;
  const uint32_t* pair_total = nullptr;
  if (dense) {
    const uint32_t qb = (uint32_t)((m + 255) / 256);
    const uint32_t *listed = nullptr, *wanted = nullptr;
    if (m >= kOrderMin && P.n >= kOrderPoints &&
        (P.last_candidates < 0.0 || P.last_candidates >= kListedCandidates)) {
      if (P.last_candidates < 0.0) {
        wanted = qs.pack_wanted;
        ProfScope ps("cells_sample", s);
        if (P.curve == SFC_CURVE_HILBERT)
          sample_cells<SFC_CURVE_HILBERT><<<1, kSampled, 0, s>>>(
              (const double2*)P.q, P.delta, m, P.occ, kListedCells, qs.pack_wanted);
        else
          sample_cells<SFC_CURVE_MORTON><<<1, kSampled, 0, s>>>(
              (const double2*)P.q, P.delta, m, P.occ, kListedCells, qs.pack_wanted);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      if ((e = order_queries(P.q, m, P.curve, P.keys, P.n, qs.perm, qs.order_scratch, s,
                             wanted)) != hipSuccess)
        return e;
      listed = qs.perm;
    }
    ProfScope ps("cells_pack", s);
#define SFC_CELLS(C, R)                                                                    \
  cells_pack<C, R><<<qb, 256, 0, s>>>((const double2*)P.q, P.delta, m, P.occ, qs.regions,  \
                                      qs.pack_cnt, qs.pack_pruned, qs.pack_flags, rec, qs.slots, \
                                      listed, wanted)
    if (P.curve == SFC_CURVE_HILBERT) {
      if (refine) SFC_CELLS(SFC_CURVE_HILBERT, true);
      else SFC_CELLS(SFC_CURVE_HILBERT, false);
    } else {
      if (refine) SFC_CELLS(SFC_CURVE_MORTON, true);
      else SFC_CELLS(SFC_CURVE_MORTON, false);
    }
#undef SFC_CELLS
    if ((e = hipGetLastError()) != hipSuccess) return e;
    pack_scan<<<1, 1024, 0, s>>>(qs.pack_cnt, qb, qs.pack_pre, qs.pack_pre + qb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    pack_move<<<qb, 256, 0, s>>>(qs.regions, qs.pack_cnt, qs.pack_pre, qs.pairs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    pairs = qs.pairs;
    pair_total = qs.pack_pre + qb;
    qs.stats_np = qb;
  }
  {
    ProfScope ps(learned ? "ranges_learned" : stree ? "ranges_stree" : "ranges_search", s);
#define SFC_RANGES(C, R, S)                                                                  \
  if (dense || dbg) SFC_RANGES_Q(C, R, S, false);                                            \
  else SFC_RANGES_Q(C, R, S, true)
#define SFC_RANGES_Q(C, R, S, Q)                                                             \
  ranges_search<C, R, S, Q><<<query_blocks(qs), 256, 0, s>>>(                                 \
      (const double2*)P.q, P.delta, m, P.keys, P.n, lv, sv, P.refine_min, P.ball,             \
      dbg ? nullptr : P.occ, pairs, pair_total, P.qset, P.set_off, P.n_sets, perm, rec,       \
      qs.slots, blk_rows, qs.blk_stat, qs.blk_rows64, qs.blk_learned, P.dbg_lo, P.dbg_hi,  \
      P.dbg_b, P.dbg_e, P.dbg_nr)
#define SFC_RANGES_R(C, R)                      \
  if (learned) {                                \
    SFC_RANGES(C, R, 1);                        \
  } else if (stree) {                           \
    SFC_RANGES(C, R, 2);                        \
  } else {                                      \
    SFC_RANGES(C, R, 0);                        \
  }
#define SFC_RANGES_C(C)                         \
  if (refine) {                                 \
    SFC_RANGES_R(C, true)                       \
  } else {                                      \
    SFC_RANGES_R(C, false)                      \
  }
    if (P.curve == SFC_CURVE_HILBERT) {
      SFC_RANGES_C(SFC_CURVE_HILBERT)
    } else {
      SFC_RANGES_C(SFC_CURVE_MORTON)
    }
#undef SFC_RANGES_C
#undef SFC_RANGES_R
#undef SFC_RANGES
#undef SFC_RANGES_Q
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (dense && (e = launch_slot_rows(qs, nullptr, qs.blk_rows, s)) != hipSuccess) return e;
  return finish_ranges(qs, P.need_rows, P.host, s);
}

// Blocks of the compaction kernels (a loop over tiles beyond this): 16384,
// 64 per CU, measured best of 4096 to 32768 (the 2^24 batch's test and write
// passes 0.968 -> 0.958 ms against 8192).
constexpr uint64_t kCompactGrid = 16384;

hipError_t launch_compact(const CompactPlan& P, const QueryScratch& qs0, hipStream_t s) {
  hipError_t e;
  QueryScratch qs = qs0;
  const uint64_t m = qs.m;
  if (m == 0) return fill_u64(P.offsets, 0, 1, s);
  // Whether the test pass may meet queries with coarser cells: known (0, 1)
  // when the caller read the batch's flag, else (-1) the pass reads it.
  const bool shifts = P.coarse != 0;
  // Rows are processed in chunks of at most kCompactChunkTiles tiles.
  // Host-sized: max_rows is the exact number of rows.  Device-sized: max_rows
  // is a capacity; each kernel reads the row count on the device, chunks past
  // it do no work, and a count above the capacity is flagged as overflow.
  const uint64_t tiles_all = (P.max_rows + kCompactTileRows - 1) / kCompactTileRows;
  const uint64_t chunk = compact_chunk_tiles();
  const uint64_t ch_tiles = tiles_all < chunk ? (tiles_all ? tiles_all : 1) : chunk;
  const uint64_t chunks = tiles_all ? (tiles_all + chunk - 1) / chunk : 1;
  CompactScratch c;
  if (!compact_carve(P.scratch, ch_tiles, &c)) return hipErrorInvalidValue;
  // write_only: the masks and unit offsets of an earlier call on the same
  // batch are still in scratch (one chunk only); run the write pass again.
  if (P.write_only && chunks != 1) return hipErrorInvalidValue;
  const uint64_t shape_rows = P.shape_rows ? P.shape_rows : P.max_rows;
  // Rows in curve order: only one chunk's hits are kept, so many chunks are
  // processed in query order.
  const bool ordered = chunks == 1 && rows_ordered(P, qs);
  const uint32_t* perm = ordered ? qs.perm : nullptr;
  const uint64_t* blk_rows = ordered ? qs.blk_place : qs.blk_rows;
  if (!P.write_only && ordered != qs.perm_made) {
    // The rows' scan so far is over the other order's workgroups.
    if (ordered && (e = order_queries(P.q, m, P.dim == 3 ? SFC_CURVE_MORTON3 : P.curve, P.keys, P.n,
                                      qs.perm, qs.order_scratch, s)) != hipSuccess)
      return e;
    uint64_t* rows = ordered ? qs.blk_place : qs.blk_rows;
    if ((e = launch_slot_rows(qs, perm, rows, s)) != hipSuccess) return e;
    if ((e = launch_rows_scan(qs, rows, qs.fused, nullptr, s)) != hipSuccess) return e;
    qs.fused = false;
  }
  const GroupSums* groups = scan_groups(qs);
  const bool fused_units = !ordered && chunks == 1 && ch_tiles * kTileUnits <= kFusedUnits;
  const uint64_t* total_dev = qs.row_off + m;
  // A batch with more rows is flagged, and none of its rows is tested.
  const uint64_t max_rows64 = P.device_sized ? P.max_rows : ~0ull;
  const uint64_t* carry = nullptr;
  int buf = 0;
  for (uint64_t ci = 0; ci < chunks; ++ci, buf ^= 1) {
    const uint64_t rbase = ci * chunk * kTileRows;
    const uint64_t nt = tiles_all - ci * chunk < chunk ? (tiles_all ? tiles_all - ci * chunk : 1)
                                                       : chunk;
    const uint64_t rend = rbase + nt * kTileRows;
    // A full chunk ends at its last tile; the last chunk at the capacity: at
    // most two rows of 32 for one of 64.
    const uint64_t row_end = ci + 1 == chunks && P.device_sized ? 2 * P.max_rows : rend;
    // A multiple of eight workgroups, so that each XCD gets its share.
    const uint32_t grid = (uint32_t)(((nt < kCompactGrid ? nt : kCompactGrid) + 7) / 8 * 8);
    uint64_t* unit_off = c.unit_off[buf];
    if (!P.write_only) {
      ProfScope ps("expand_rows", s);
#define SFC_EXPAND(K, F)                                                                     \
  expand_rows<K, F><<<query_blocks(qs), 256, 0, s>>>(                                        \
      qs.row_off, qs.slots, perm, blk_rows, qs.blk_off, groups, stats_of(qs), qs.status, m,  \
      qs.ss, rbase, row_end, max_rows64, P.reject, c.meta, c.info)
      switch (slots_per_thread(qs)) {
        case 1: if (qs.fused) SFC_EXPAND(1, true); else SFC_EXPAND(1, false); break;
        case 2: if (qs.fused) SFC_EXPAND(2, true); else SFC_EXPAND(2, false); break;
        default: if (qs.fused) SFC_EXPAND(4, true); else SFC_EXPAND(4, false); break;
      }
#undef SFC_EXPAND
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (!P.write_only) {
      ProfScope ps("compact_test", s);
#define SFC_TEST_K(R, I, E, D, C, W, K)                                                    \
  compact_test<R, I, E, D, C, W, K><<<grid, 256, 0, s>>>(                                  \
      P.q, P.delta, m, P.pts ? P.pts : P.pts_in, P.pts ? nullptr : P.ids, P.cells, qs.rec, \
      c.meta, total_dev, rbase, row_end, c.masks, c.info, c.unit_hits, qs.status, P.ins, P.era)
#define SFC_TEST_W(R, I, E, D, C, W)                                                       \
  if (C && shifts) SFC_TEST_K(R, I, E, D, C, W, C);                                        \
  else SFC_TEST_K(R, I, E, D, C, W, false)
#define SFC_TEST(R, I, E, D, C)                                                            \
  if (P.window) SFC_TEST_W(R, I, E, D, C, true);                                           \
  else SFC_TEST_W(R, I, E, D, C, false)
#define SFC_TEST_SHAPES(E, D, C)              \
  switch (test_variant(shape_rows)) {         \
    case 1: SFC_TEST(4, 4, E, D, C); break;   \
    case 2: SFC_TEST(8, 2, E, D, C); break;   \
    case 3: SFC_TEST(2, 8, E, D, C); break;   \
    case 4: SFC_TEST(1, 16, E, D, C); break;  \
    default: SFC_TEST(16, 1, E, D, C); break; \
  }
      if (P.ins && (P.cells || P.dim == 3)) return hipErrorInvalidValue;   // never kept together
      if (P.dim == 3) {
        if (P.cells) {
          SFC_TEST_SHAPES(false, 3, true)
        } else {
          SFC_TEST_SHAPES(false, 3, false)
        }
      } else if (P.cells) {
        SFC_TEST_SHAPES(false, 2, true)
      } else if (P.ins) {
        SFC_TEST_SHAPES(true, 2, false)
      } else {
        SFC_TEST_SHAPES(false, 2, false)
      }
#undef SFC_TEST_SHAPES
#undef SFC_TEST
#undef SFC_TEST_W
#undef SFC_TEST_K
      if ((e = hipGetLastError()) != hipSuccess) return e;
      if (!fused_units &&
          (e = scan_excl_dev(c.unit_hits, unit_off, &qs.status->units, nt * kTileUnits, carry,
                             c.scan_tmp, s)) != hipSuccess)
        return e;
    }
    if (ordered) {
      ProfScope ps("query_offsets", s);
      const uint32_t qb = (uint32_t)((m + 255) / 256);
      if (!P.write_only) {
        query_hits<<<qb, 256, 0, s>>>(qs.row_off, m, qs.status, c.info, unit_off, qs.perm,
                                      qs.qhits, qs.out_base);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      if ((e = scan_excl(qs.qhits, P.offsets, m, nullptr, qs.scan_tmp, s)) != hipSuccess) return e;
      if (!P.write_only) {
        place_rows<<<qb, 256, 0, s>>>(P.offsets, m, qs.out_base);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
    }
    {
      ProfScope ps("compact_write", s);
      const uint32_t extra = ordered ? 0 : fill_blocks(m + 1);
#define SFC_WRITE(O, F)                                                                      \
  compact_write_out<O, F><<<grid + extra, 256, 0, s>>>(                                       \
      P.ids, c.meta, qs.row_off, m, rbase, rend, row_end, c.masks, c.info, c.unit_hits,       \
      unit_off, qs.out_base, grid, P.out_ids, P.cap, chunks == 1, P.offsets, qs.status,       \
      P.host, P.flags_out)
      if (ordered) SFC_WRITE(true, false);
      else if (fused_units) SFC_WRITE(false, true);
      else SFC_WRITE(false, false);
#undef SFC_WRITE
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // The chunk's total, read by the next chunk's scan.  A chunk has tiles
    // only when every chunk before it was full, so this slot is always
    // written when it is consumed.
    carry = unit_off + nt * kTileUnits;
  }
  return hipSuccess;
}

}  // namespace sfc
