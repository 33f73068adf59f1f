// Static search tree over the sorted keys (Sec. 2.1 "Storing P twice": the
// keys are searched through a static B-tree whose lowest layer is the sorted
// key array itself).  Our layout: layer 0 is the key array; layer k+1 holds
// the first key of every block of kStreeFan consecutive entries of layer k
// (a 128-byte line), so layer k+1[b] = keys[b * kStreeFan^(k+1)].  A layer of
// at most kStreeFan entries is the top.
//
// Counting the entries of layer 0 below x: let c be the number of entries of
// layer k+1 below x, i.e. of blocks of layer k whose first entry is below x.
// All entries of the blocks before block c-1 are then below x too, and none
// after it, so the count in layer k is kStreeFan * (c - 1) plus the count
// inside block c-1 (and 0 when c = 0).  One line per layer, top down.  The
// same holds with "at most x" for the upper end of a key interval, so a key
// interval [lo, hi] maps to the index range [#(< lo), #(<= hi)), equal to
// std::lower_bound / std::upper_bound over the keys.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sfc {

constexpr int kStreeFan = 16;          // entries per block: one 128-byte line of u64 keys
constexpr int kStreeMaxLayers = 9;     // 2^32 keys: layers of 2^32, 2^28, ..., 16

// Device view: layer[0] is the key array (16-byte aligned), layers 1..top
// live in one buffer, each 256-byte aligned.
struct StreeView {
  const uint64_t* layer[kStreeMaxLayers];
  uint64_t size[kStreeMaxLayers];
  int top;
};

// The last entries of the first three quarters of the block at `base` of a
// layer of `size` entries (2^64 - 1 past its end).
__device__ __forceinline__ void stree_pivots(const uint64_t* __restrict__ layer, uint32_t size,
                                             uint32_t base, uint64_t (&v)[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const uint32_t at = base + 4 * i + 3;
    v[i] = layer[at < size ? at : size - 1];
  }
}

// Entries among the four at `at` (in a layer of `size` entries) that are below x
// (LE: at most x).
template <bool LE>
__device__ __forceinline__ uint32_t stree_count4(const uint64_t (&w)[4], uint32_t size, uint32_t at,
                                                 uint64_t x) {
  uint32_t c = 0;
#pragma unroll
  for (int t = 0; t < 4; ++t) c += (LE ? w[t] <= x : w[t] < x) && at + t < size ? 1u : 0u;
  return c;
}
__device__ __forceinline__ void stree_load4(const uint64_t* __restrict__ layer, uint32_t size,
                                            uint32_t at, uint64_t (&w)[4]) {
  if (size - at >= 4) {
    const ulonglong2* p = (const ulonglong2*)(layer + at);
    const ulonglong2 a = p[0], b = p[1];
    w[0] = a.x;
    w[1] = a.y;
    w[2] = b.x;
    w[3] = b.y;
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t) w[t] = layer[at + t < size ? at + t : size - 1];
  }
}

// The index range [b, e) of the key interval [lo, hi], lo <= hi: both descents
// run level by level together.  On the GPU a lane's loads, each a cache lookup,
// cost as much as the lines they bring in.  So a block takes five: the last
// entries of its quarters, then the quarter that holds the count (eight 16-byte
// loads brought the whole line: 1.06 ms for 2^20 refined queries over 2^24 points
// in space, this 1.00, memory's 6 TB/s of lines its limit); and the lower end,
// which is in the upper end's block on most layers, takes loads of its own only
// where it is not.
__device__ __forceinline__ void stree_range(const StreeView& v, uint64_t lo, uint64_t hi,
                                            uint64_t& b, uint64_t& e) {
  uint32_t cb = 1, ce = 1;   // the top layer is one block (indices fit 32 bits, as ids do)
  if (v.size[0] == 0) cb = ce = 0;
  for (int k = v.top; k >= 0; --k) {
    const uint64_t* __restrict__ L = v.layer[k];
    const uint32_t sz = (uint32_t)v.size[k];
    if (ce == 0) break;      // then cb is 0 too: no entry is at most hi
    const uint32_t be = (ce - 1) * kStreeFan, bb = cb > 0 ? (cb - 1) * kStreeFan : be;
    uint64_t pe[3], pb[3];
    stree_pivots(L, sz, be, pe);
#pragma unroll
    for (int i = 0; i < 3; ++i) pb[i] = pe[i];
    if (bb != be) stree_pivots(L, sz, bb, pb);
    uint32_t ae = be, ab = bb;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      ae += pe[i] <= hi && be + 4 * i + 3 < sz ? 4u : 0u;
      ab += pb[i] < lo && bb + 4 * i + 3 < sz ? 4u : 0u;
    }
    uint64_t we[4], wb[4];
    stree_load4(L, sz, ae, we);
#pragma unroll
    for (int i = 0; i < 4; ++i) wb[i] = we[i];
    if (ab != ae) stree_load4(L, sz, ab, wb);
    ce = ae + stree_count4<true>(we, sz, ae, hi);
    if (cb > 0) cb = ab + stree_count4<false>(wb, sz, ab, lo);
  }
  b = cb;
  e = ce;
}

// Host: bytes of layers 1..top for n keys, and the view over keys and buf.
size_t stree_bytes(uint64_t n);
StreeView stree_view(const uint64_t* keys, uint64_t n, void* buf);
// Writes layers 1..top of v from its layer 0.
hipError_t stree_build(const StreeView& v, hipStream_t s);

}  // namespace sfc
