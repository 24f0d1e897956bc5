// Where the fused conv/FC1 kernels of small batches find a patch's rows (paper
// §2.1: the patch of hit (w, t) holds image[w - 24 + r][t - 24 + c], 0 outside
// the plane).  They read the fp32 rows of the plane image, or of a pre-cut
// patch, themselves: no patch is written to memory and read back, and the
// gather's launch is saved, about 8 us of a call of 128 hits.
//
// A patch's rows are described by 16 bytes: the address of its pixel (0, 0)
// (which may lie outside the image), the image's row pitch, and the ranges of
// patch rows and columns that are inside the plane.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"

namespace pointid {

typedef float rowx4 __attribute__((ext_vector_type(4)));
typedef float rowx4_u __attribute__((ext_vector_type(4), aligned(4)));

// Row descriptor as a uint4: x, y the address, z the row pitch in pixels,
// w = r_lo | r_hi << 8 | c_lo << 16 | c_hi << 24 (half-open ranges; 0: no pixel).
__device__ __forceinline__ uint4 row_desc(uint64_t base, uint32_t pitch, uint32_t ranges) {
  return make_uint4((uint32_t)base, (uint32_t)(base >> 32), pitch, ranges);
}

// Pre-cut patch p of fp32 patches [n][48][48].
__device__ __forceinline__ uint4 patch_row_desc(const float* patches, int64_t p) {
  return row_desc(reinterpret_cast<uint64_t>(patches + p * kPatchPix), kPatch,
                  (uint32_t)kPatch << 8 | (uint32_t)kPatch << 24);
}

// Hit (plane, wire w, column t) on the planes of `planes`; a plane out of
// range has no pixel.
__device__ __forceinline__ uint4 hit_row_desc(const PlaneTable& planes, int plane, int w, int t) {
  if (plane < 0 || plane >= planes.n) return make_uint4(0, 0, 0, 0);
  const int64_t W = planes.p[plane].n_wires, T = planes.p[plane].n_ticks;
  const int64_t w0 = (int64_t)w - kHalf, t0 = (int64_t)t - kHalf;
  auto clamp48 = [](int64_t v) { return (uint32_t)(v < 0 ? 0 : (v > kPatch ? kPatch : v)); };
  const uint32_t r_lo = clamp48(-w0), r_hi = clamp48(W - w0);
  const uint32_t c_lo = clamp48(-t0), c_hi = clamp48(T - t0);
  if (r_lo >= r_hi || c_lo >= c_hi) return make_uint4(0, 0, 0, 0);
  const uint64_t base = reinterpret_cast<uint64_t>(planes.p[plane].image) + 4 * (uint64_t)(w0 * T + t0);
  return row_desc(base, (uint32_t)T, r_lo | r_hi << 8 | c_lo << 16 | c_hi << 24);
}

// Patch i of a batch of requests (one request when tab.n == 1; unused entries
// of start hold INT64_MAX); `div` ticks per image column.
__device__ __forceinline__ uint4 request_row_desc(const PlaneTable& planes, const RequestTable& tab,
                                                  int div, int64_t i) {
  // the request holding patch i: the starts at or before it, all table reads scalar
  int r = 0;
  if (tab.n > 1) {
#pragma unroll
    for (int k = 1; k < kMaxRequests; ++k) r += tab.start[k] <= i ? 1 : 0;
  }
  const int64_t j = i - tab.start[r];
  int plane = tab.plane[r], w, t;
  if (plane >= 0) {
    const int32_t* h = tab.hits[r] + 2 * j;
    w = h[0];
    t = h[1];
  } else {
    const int32_t* h = tab.hits[r] + 3 * j;
    plane = h[0];
    w = h[1];
    t = h[2];
  }
  if (div > 1) {                             // floor(t / div)
    const int q = t / div;
    t = (q * div != t && t < 0) ? q - 1 : q;
  }
  return hit_row_desc(planes, plane, w, t);
}

// Pixels 4h .. 4h + 3 of row r of the patch described by d, in two halves so
// that a kernel can do other work while they arrive.
//
// row_chunk_load issues one 16-byte load (at a 4-byte aligned address) without
// a branch, so that the loads of several chunks are in flight together: the
// chunk's own address where all four pixels are inside the plane, else `safe`,
// any 16 readable bytes.  Lanes take consecutive chunks, so that a load
// instruction touches each cache line of a patch row once.
// Streamed: non-temporal, so the rows do not push the FC1 weights out of L2.
constexpr int kRowChunks = kPatch / 4;
constexpr uint32_t kRowWhole = 0, kRowPart = 1, kRowNone = 2;   // pixels of a chunk inside the plane
__device__ __forceinline__ uint64_t row_chunk_addr(const uint4& d, int r, int h) {
  const uint64_t base = ((uint64_t)d.y << 32) | d.x;
  return base + 4 * ((uint64_t)(uint32_t)r * d.z + 4u * (uint32_t)h);
}
// A descriptor out of LDS, all of it at once (used on conditions, the compiler
// would read its parts one after the other behind branches).
__device__ __forceinline__ uint4 desc_from_lds(const uint4* p) {
  uint4 d = *p;
  asm volatile("" : "+v"(d.x), "+v"(d.y), "+v"(d.z), "+v"(d.w));
  return d;
}
__device__ __forceinline__ rowx4 row_chunk_load(const uint4& d, int r, int h, const void* safe,
                                                uint32_t* kind) {
  typedef __attribute__((address_space(1))) const rowx4_u* gvec;
  const uint32_t r_lo = d.w & 255u, r_hi = (d.w >> 8) & 255u;
  const uint32_t c = 4u * (uint32_t)h, c_lo = (d.w >> 16) & 255u, c_hi = d.w >> 24;
  const bool any = ((uint32_t)r - r_lo < r_hi - r_lo) & (c < c_hi) & (c + 4 > c_lo);
  const bool whole = any & (c >= c_lo) & (c + 4 <= c_hi);
  *kind = whole ? kRowWhole : any ? kRowPart : kRowNone;
  uint64_t at = row_chunk_addr(d, r, h);
  asm volatile("" : "+v"(at));               // computed by every lane: a select, not a branch
  at = whole ? at : reinterpret_cast<uint64_t>(safe);
  return __builtin_nontemporal_load((gvec)at);
}
// The chunk's pixels from what row_chunk_load gave: 0 outside the plane; a
// chunk across the plane's first or last column (hits near it only) is read
// here, pixel by pixel, from its descriptor.
__device__ __forceinline__ rowx4 row_chunk_finish(const uint4* desc, int r, int h, rowx4 v, uint32_t kind) {
  typedef __attribute__((address_space(1))) const float* gptr;
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = kind == kRowWhole ? v[j] : 0.f;
  if (kind == kRowPart) {
    // (the values are made to arrive inside the branch: behind it the wait for
    // them would hold up every wave's other loads)
    const uint4 d = *desc;
    const uint32_t c = 4u * (uint32_t)h, c_lo = (d.w >> 16) & 255u, c_hi = d.w >> 24;
    const gptr at = (gptr)row_chunk_addr(d, r, h);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (c + j >= c_lo && c + j < c_hi) v[j] = at[j];
    asm volatile("" : "+v"(v));
  }
  return v;
}

// Where the patches of a launch come from, on the host: pre-cut fp32 patches,
// 16-bit patches made by the gather, or hits on planes.
struct RowInput {
  const float* patches = nullptr;
  const uint16_t* patches16 = nullptr;
  const PlaneTable* planes = nullptr;
  const RequestTable* reqs = nullptr;
  int div = 1;                               // ticks per image column
};

// In a kernel that resolves the hits itself: patches when given, else hits.
struct HitSource {
  const float* patches;
  int64_t n;
  int32_t div;
  PlaneTable planes;
  RequestTable reqs;
  __device__ __forceinline__ uint4 get(int64_t p) const {
    if (p >= n) return make_uint4(0, 0, 0, 0);       // past the batch: no pixel, never stored
    return patches ? patch_row_desc(patches, p) : request_row_desc(planes, reqs, div, p);
  }
};
// Pre-cut patches alone, whose rows need no descriptor.
struct PatchSource {
  const float* patches;
  int64_t n;
};
inline HitSource hit_source(const RowInput& in, int64_t n) {
  HitSource s = {};
  s.patches = in.patches;
  s.n = n;
  s.div = in.div;
  if (!in.patches) {
    s.planes = *in.planes;
    s.reqs = *in.reqs;
  }
  return s;
}

}  // namespace pointid
