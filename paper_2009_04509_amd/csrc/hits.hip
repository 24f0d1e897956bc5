// Hit finding on deconvolved plane images (paper §2.1: the reconstruction
// finds wire hits on the deconvolved waveforms before they are classified; the
// paper names no algorithm).  A tick t of a wire's waveform x is a hit when
//   x[t] > threshold,  x[t] > x[t-1]  and  x[t] >= x[t+1],
// where ticks outside the waveform count as minus infinity, so a plateau gives
// one hit at its first tick.  Comparisons are exact fp32 comparisons, so the
// result is bit-exact.  Hits come out as (plane, wire, tick) in plane, then
// wire, then tick order: the same order on every run, whatever the launch.
//
// The waveforms are cut into steps of 256 ticks (one wire each), numbered in
// output order, and every wave ("worker") owns one contiguous range of steps,
// so all workers have the same amount of image to read whatever the plane
// shapes.  Two launches, each a plain pass (no atomics, no waits between
// blocks):
//   mask   per step, 4 consecutive ticks per lane (one 16-byte load), the
//          neighbours from the adjacent lanes and, at the step's two ends,
//          one extra value; the step's hit bits are packed in tick order (8
//          words, 32 B), the worker's and the block's hit counts stored at the end;
//   emit   a block of the same 4 workers: its first output index is the sum of
//          the counts of the blocks before it (at most 2,048 words, a few loads
//          per thread; a scan launch of its own took 8.9 us).  A lane takes one
//          hit: the step from a binary search in the steps' prefix sums, the
//          word and the bit from bit counts, and consecutive lanes store
//          consecutive rows.  (A pass with one step per wave at a time, whatever
//          its few hits, was bound by instruction issue: 39.6 us on the event.)
//          Where a wave's steps hold 32 hits or more each, a step at a time costs
//          less than the searches: lanes take 4 ticks each, and the step's ticks
//          are put in order through LDS (event's planes, us per call with the
//          searches and a step at a time: every local maximum, 85 of 256 ticks, 189
//          and 155; those above 1.2 sigma of the noise, 26 a step, 122 and 115;
//          above 1.6, 13 a step, 108 and 112; above 4, signal only, 82 and 90).
// The image is read once (the bits are 1/32 of it), so the whole call is bound
// by HBM reads of the image.
#include "pointid.h"
#include "internal.h"

namespace pointid {
namespace {

constexpr int kMaskWaves = 4;             // workers per mask block
constexpr int kUnroll = 8;                // steps whose loads are in flight together

// Position of a step: plane p, wire `row`, step s along the wire, with plane
// p's sizes and the wire's first tick cached (reloaded only when the cursor
// enters the next plane).
struct Cursor {
  int p, row, s;
  int per_row, n_wires, T;
  const float* x;                                // tick 0 of wire `row`
};

__device__ __forceinline__ void enter_plane(const PlaneTable& planes, const HitSteps& st,
                                            Cursor& c) {
  c.per_row = st.per_row[c.p];
  c.n_wires = planes.p[c.p].n_wires;
  c.T = planes.p[c.p].n_ticks;
  c.x = planes.p[c.p].image + (int64_t)c.row * c.T;
}

__device__ __forceinline__ Cursor locate(const PlaneTable& planes, const HitSteps& st, int64_t g) {
  int p = 0, hi = st.n - 1;                      // last plane starting at or before g
  while (p < hi) {
    const int mid = (p + hi + 1) >> 1;
    if (st.step0[mid] <= g) p = mid;
    else hi = mid - 1;
  }
  const int64_t local = g - st.step0[p];
  const int64_t per_row = st.per_row[p];
  Cursor c;
  c.p = p;
  c.row = (int)(local / per_row);
  c.s = (int)(local - (int64_t)c.row * per_row);
  enter_plane(planes, st, c);
  return c;
}

__device__ __forceinline__ void advance(const PlaneTable& planes, const HitSteps& st, Cursor& c) {
  if (++c.s == c.per_row) {
    c.s = 0;
    c.x += c.T;
    if (++c.row == c.n_wires) {
      c.row = 0;
      if (++c.p < st.n) enter_plane(planes, st, c);
    }
  }
}

template <bool kVec>
__global__ __launch_bounds__(64 * kMaskWaves) void hits_mask_kernel(PlaneTable planes, HitSteps st,
                                                                    float thr,
                                                                    uint32_t* __restrict__ mask,
                                                                    int32_t* __restrict__ counts,
                                                                    int32_t* __restrict__ block_counts) {
  __shared__ int32_t wave_counts[kMaskWaves];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t w = (int64_t)blockIdx.x * kMaskWaves + wave;
  const float ninf = -__builtin_huge_valf();
  const int64_t total = st.step0[st.n];
  int64_t g = w * st.per;
  // (a wave past the last worker has no steps)
  const int64_t end = w >= st.workers ? g : g + st.per < total ? g + st.per : total;
  Cursor c = {};
  if (g < end) c = locate(planes, st, g);
  int32_t count = 0;                                     // this lane's hits
  for (; g < end; g += kUnroll) {
    float v[kUnroll][4], edge[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const bool live = g + u < end;                     // wave-uniform
      const int64_t T = c.T;
      const float* x = c.x;
      const int64_t t0 = (int64_t)c.s * kHitStep + 4 * lane;
      if constexpr (kVec) {
        if (live && t0 < T) {                             // T % 4 == 0: all 4 inside
          const float4 q = *reinterpret_cast<const float4*>(x + t0);
          v[u][0] = q.x;
          v[u][1] = q.y;
          v[u][2] = q.z;
          v[u][3] = q.w;
        } else {
          v[u][0] = v[u][1] = v[u][2] = v[u][3] = ninf;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[u][j] = (live && t0 + j < T) ? x[t0 + j] : ninf;
      }
      // lane 0 needs the tick before the step, lane 63 the tick after it
      const int64_t te = lane == 0 ? (int64_t)c.s * kHitStep - 1 : ((int64_t)c.s + 1) * kHitStep;
      edge[u] = (live && (lane == 0 || lane == 63) && te >= 0 && te < T) ? x[te] : ninf;
      if (live) advance(planes, st, c);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      if (g + u >= end) break;                           // wave-uniform
      float before = __shfl_up(v[u][3], 1);
      float after = __shfl_down(v[u][0], 1);
      if (lane == 0) before = edge[u];
      if (lane == 63) after = edge[u];
      const float* a = v[u];
      uint32_t x = (a[0] > thr && a[0] > before && a[0] >= a[1] ? 1u : 0u) |
                   (a[1] > thr && a[1] > a[0] && a[1] >= a[2] ? 2u : 0u) |
                   (a[2] > thr && a[2] > a[1] && a[2] >= a[3] ? 4u : 0u) |
                   (a[3] > thr && a[3] > a[2] && a[3] >= after ? 8u : 0u);
      count += __popc(x);
      // the 4 bits of 8 lanes into one word: lanes 1, 2, then 4 further on
      // (row_shl: within rows of 16 lanes)
      x |= __builtin_amdgcn_update_dpp(0, x, 0x101, 0xf, 0xf, true) << 4;
      x |= __builtin_amdgcn_update_dpp(0, x, 0x102, 0xf, 0xf, true) << 8;
      x |= __builtin_amdgcn_update_dpp(0, x, 0x104, 0xf, 0xf, true) << 16;
      if ((lane & 7) == 0) mask[(g + u) * 8 + (lane >> 3)] = x;
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) count += __shfl_xor(count, d);
  if (lane == 0) {
    wave_counts[wave] = count;
    if (w < st.workers) counts[w] = count;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t sum = 0;
    for (int k = 0; k < kMaskWaves; ++k) sum += wave_counts[k];
    block_counts[blockIdx.x] = sum;
  }
}

// Inclusive prefix sum over the 64 lanes.
__device__ __forceinline__ int wave_incl_scan(int x, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  return x;
}

// Keeps the compiler from moving LDS accesses across this point.  A wave's
// LDS instructions execute in issue order, so a lane reading what another lane
// of the same wave wrote earlier needs no wait (the waves of an emit block
// share no staging).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}

// Position of the r-th set bit (r from 0) of x.
__device__ __forceinline__ int nth_bit(uint32_t x, int r) {
  int pos = 0;
#pragma unroll
  for (int width = 16; width > 0; width >>= 1) {
    const int below = __popc(x & ((1u << width) - 1));
    const bool up = r >= below;
    r -= up ? below : 0;
    x >>= up ? width : 0;
    pos += up ? width : 0;
  }
  return pos;
}

// 64 steps of one wave: their first hit, bits, plane, wire and first tick; a
// step's hits in order (at most every second tick).
constexpr int kDenseStep = 32;
struct EmitStage {
  int32_t start[64];
  uint32_t bits[64][8];
  int32_t plane[64], row[64], tick[64];
  int32_t order[kHitStep / 2];
};

__global__ __launch_bounds__(64 * kMaskWaves) void hits_emit_kernel(
    PlaneTable planes, HitSteps st, const uint32_t* __restrict__ mask,
    const int32_t* __restrict__ counts, const int32_t* __restrict__ block_counts,
    int32_t* __restrict__ hits, int64_t capacity, int64_t* __restrict__ n_found) {
  __shared__ EmitStage stages[kMaskWaves];
  __shared__ int64_t wave_sums[kMaskWaves];
  constexpr int kPer = kHitMaxWorkers / kMaskWaves / (64 * kMaskWaves);   // block counts per thread
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int64_t w = (int64_t)blockIdx.x * kMaskWaves + wave;
  // hits of the blocks before this one
  const bool last = blockIdx.x + 1 == gridDim.x;
  const int32_t own = block_counts[blockIdx.x];
  if (own == 0 && !last) return;                         // block-uniform
  int64_t sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = threadIdx.x + k * 64 * kMaskWaves;
    sum += i < (int)blockIdx.x ? block_counts[i] : 0;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
  if (lane == 0) wave_sums[wave] = sum;
  __syncthreads();
  int64_t base = 0;
#pragma unroll
  for (int k = 0; k < kMaskWaves; ++k) base += wave_sums[k];
  if (last && threadIdx.x == 0) *n_found = base + own;
  if (w >= st.workers) return;                           // wave-uniform; no barrier below
  for (int k = 0; k < wave; ++k) base += counts[w - wave + k];
  if (counts[w] == 0 || base >= capacity) return;

  EmitStage& sg = stages[wave];
  const int64_t total = st.step0[st.n];
  const int64_t g0 = w * st.per;
  const int64_t g1 = g0 + st.per < total ? g0 + st.per : total;
  int p0 = 0, hi = st.n - 1;                             // the plane of step g0
  while (p0 < hi) {
    const int mid = (p0 + hi + 1) >> 1;
    if (st.step0[mid] <= g0) p0 = mid;
    else hi = mid - 1;
  }
  for (int64_t c = g0; c < g1 && base < capacity; c += 64) {
    const int64_t g = c + lane;
    // lane k: step c + k
    uint4 lo = make_uint4(0, 0, 0, 0), up = lo;
    if (g < g1) {
      lo = reinterpret_cast<const uint4*>(mask)[2 * g];
      up = reinterpret_cast<const uint4*>(mask)[2 * g + 1];
    }
    const int n = __popc(lo.x) + __popc(lo.y) + __popc(lo.z) + __popc(lo.w) + __popc(up.x) +
                  __popc(up.y) + __popc(up.z) + __popc(up.w);
    const int incl = wave_incl_scan(n, lane);
    const int found = __builtin_amdgcn_readlane(incl, 63);
    int p = p0;
    int64_t first = st.step0[p0];
    int per_row = st.per_row[p0];
    for (int q = p0 + 1; q < st.n && st.step0[q] <= c + 63; ++q) {   // planes that start in the chunk
      if (g >= st.step0[q]) {
        p = q;
        first = st.step0[q];
        per_row = st.per_row[q];
      }
    }
    const int64_t local = g - first;
    const int row = (int)(local / per_row);
    sg.start[lane] = incl - n;
    reinterpret_cast<uint4*>(sg.bits[lane])[0] = lo;
    reinterpret_cast<uint4*>(sg.bits[lane])[1] = up;
    sg.plane[lane] = p;
    sg.row[lane] = row;
    sg.tick[lane] = (int)(local - (int64_t)row * per_row) * kHitStep;
    p0 = __builtin_amdgcn_readlane(p, 63);
    wave_lds_order();
    const int lim = (int)(found < capacity - base ? found : capacity - base);
    const int live = (int)(g1 - c < 64 ? g1 - c : 64);
    if (found >= kDenseStep * live) {
      // lane l with the ticks 4l .. 4l + 3 of a step
      for (int k = 0; k < live; ++k) {                   // (wave-uniform)
        const uint32_t x = sg.bits[k][lane >> 3] >> (4 * (lane & 7)) & 15u;
        const int first = __builtin_amdgcn_readfirstlane(sg.start[k]);
        if (first >= lim) break;
        const int next = k < live - 1 ? __builtin_amdgcn_readfirstlane(sg.start[k + 1]) : found;
        int pos = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint64_t b = __ballot((x >> j & 1u) != 0);
          pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, pos));
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (x >> j & 1u) sg.order[pos++] = 4 * lane + j;
        wave_lds_order();
        const int n_k = (next < lim ? next : lim) - first;
        const int p = sg.plane[k], w = sg.row[k], t = sg.tick[k];
        for (int i = lane; i < n_k; i += 64) {
          int32_t* o = hits + 3 * (base + first + i);
          o[0] = p;
          o[1] = w;
          o[2] = t + sg.order[i];
        }
        wave_lds_order();
      }
    } else {
      for (int i = lane; i < lim; i += 64) {
        int k = 0;                                         // the last step that starts at or before hit i
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) k += sg.start[k + d] <= i ? d : 0;
        int r = i - sg.start[k];
        uint32_t x = 0;
        int word = 0;
        bool open = true;
#pragma unroll
        for (int j = 0; j < 8; ++j) {                      // the word holding its r-th hit
          const uint32_t v = sg.bits[k][j];
          const int m = __popc(v);
          const bool here = open && r < m;
          x = here ? v : x;
          word = here ? j : word;
          open = open && !here;
          r -= open ? m : 0;
        }
        int32_t* o = hits + 3 * (base + i);
        o[0] = sg.plane[k];
        o[1] = sg.row[k];
        o[2] = sg.tick[k] + 32 * word + nth_bit(x, r);
      }
    }
    wave_lds_order();
    base += found;
  }
}

}  // namespace

void hit_steps(const PlaneTable& planes, HitSteps* st) {
  st->n = planes.n;
  st->step0[0] = 0;
  for (int i = 0; i < planes.n; ++i) {
    st->per_row[i] = (int32_t)(((int64_t)planes.p[i].n_ticks + kHitStep - 1) / kHitStep);
    st->step0[i + 1] = st->step0[i] + (int64_t)planes.p[i].n_wires * st->per_row[i];
  }
  const int64_t total = st->step0[planes.n];
  st->per = (total + kHitMaxWorkers - 1) / kHitMaxWorkers;
  st->workers = (int32_t)((total + st->per - 1) / st->per);
}

int hit_blocks(const HitSteps& st) { return (st.workers + kMaskWaves - 1) / kMaskWaves; }

hipError_t launch_hits_mask(const PlaneTable& planes, const HitSteps& st, float threshold,
                            uint32_t* mask, int32_t* counts, int32_t* block_counts,
                            hipStream_t stream) {
  bool vec = true;
  for (int i = 0; i < planes.n; ++i)
    vec = vec && (reinterpret_cast<uintptr_t>(planes.p[i].image) & 15) == 0 &&
          planes.p[i].n_ticks % 4 == 0;
  const dim3 grid((unsigned)hit_blocks(st));
  if (vec)
    return launch_kernel(hits_mask_kernel<true>, grid, dim3(64 * kMaskWaves), 0, stream, planes, st,
                         threshold, mask, counts, block_counts);
  return launch_kernel(hits_mask_kernel<false>, grid, dim3(64 * kMaskWaves), 0, stream, planes, st,
                       threshold, mask, counts, block_counts);
}

hipError_t launch_hits_emit(const PlaneTable& planes, const HitSteps& st, const uint32_t* mask,
                            const int32_t* counts, const int32_t* block_counts, int32_t* hits,
                            int64_t capacity, int64_t* n_found, hipStream_t stream) {
  return launch_kernel(hits_emit_kernel, dim3((unsigned)hit_blocks(st)), dim3(64 * kMaskWaves), 0, stream,
                       planes, st, mask, counts, block_counts, hits, capacity, n_found);
}

}  // namespace pointid
