// Fused conv 5x5 (1->48) + ReLU + FC1 (92928->128) of the fp32 path, paper §2.2,
// on bf16 MFMAs (v_mfma_f32_16x16x32_bf16).  The conv maps exist only in
// registers, and the patch rows are read from the plane images or the pre-cut
// patches themselves (rows.h): no patch is written and read back.
//
// Arithmetic.  Every fp32 operand (pixel, filter, map value, FC1 weight) is
// taken as the exact sum of three bf16 values, high + middle + low, each the rest
// rounded to nearest, and a product as the six of its nine partial products
// that reach fp32's precision: hh, hm, mh, mm, hl, lh.  Each partial product is
// exact and all are added in fp32 MFMA accumulators; what is left out is below
// 2^-24.2 of a product (2^-27.5 in the mean square), less than fp32 rounds off a
// product (2^-24 and 2^-25.2).  The bf16 MFMA runs at 16 times
// the rate of the fp32 one, so six of them take 3/8 of its time (event of 50,000
// hits: 12.1 ms per call with fp32 MFMAs, 6.0 to 6.3 here).  Sums come out no less
// precise: against the network in 64 bits the event's scores are off by a relative
// 1.7e-6 (fp32 MFMAs: 2.1e-6), those of 235 pre-cut patches by 5.2e-7 (5.6e-7),
// because a K = 32 MFMA rounds its accumulator once per 32 inputs.
//
// Map positions go in pairs (x, x+1), x even, in 8 contiguous ranges (split-K)
// of 8 interleaved position groups, one per wave (wave g takes the pairs
// 8k + g of a range).  The 5x6 window of a pair (30 pixels; slot 30 is 1.0 for
// the bias) is one K = 32 conv operand per part; operand layouts, the two conv
// tiles that feed a K-step and the 3 K-steps of a pair are those of
// conv_fc1_16.hip.  Per K-step a wave computes the conv of each 16-patch tile
// (2 x 6 MFMAs), splits the ReLU'd maps into three FC1 operands in place, and
// runs 6 MFMAs per output tile and patch tile, two accumulators' six in turn.  The FC1 weights are packed at create, [pair][K-step][16 outputs][part]:
// a fragment feeds 2 MFMAs per patch tile, and a ring of register sets holds
// the next few output tiles' fragments, each set reloaded as soon as its MFMAs
// have issued.
//
// A wave needs no other wave's results before the final reduction, so the two
// waves of a SIMD run freely, one's conversions behind the other's MFMAs; the
// block meets only where a new patch row goes into the LDS ring (6 rows, the
// most that one step of 8 pairs needs, in three bf16 planes).  The row's loads
// are issued a K-step before that.
//
// A block takes 64 or 32 patches and one range; a patch's sums are one chain of
// MFMAs per range and group and a fixed tree over the groups, whatever the shape
// of the block.  Small batches share the 128 outputs over 2 or 4 blocks
// (`kParts`; each computes the conv).
//
// Range.  A finite pixel that could take a conv sum past a quarter of fp32's
// range, an infinite one or a NaN (ConvF32::limit: none of them occurs in charge
// images), and FC1 sums that are not finite, have no place in three parts: the
// block computes the sums of such a patch (for sums, those of their 16 outputs) again
// in plain fp32, product by product, so that infinities, NaNs and overflows come out as
// fp32 arithmetic gives them, whatever the shape of the block.
#include <algorithm>
#include <cmath>

#include "internal.h"
#include "op16.h"
#include "rows.h"

namespace pointid {
namespace {

constexpr int kWaves = 8;                     // position groups
constexpr int kThreads = kWaves * 64;
constexpr int kSplits = 8;                    // position ranges
constexpr int kMTiles = kFc1Out / 16;         // 16-output tiles
constexpr int kPairsPerRow = kFm / 2;         // 22
constexpr int kPairs = kPos / 2;              // 968
constexpr int kQ = 3;                         // K-steps per pair
constexpr int kParts3 = kF32Parts;            // bf16 parts of an fp32 value: high, middle, low
constexpr int kRing = 6;                      // patch rows in LDS
constexpr int kRP = 26;                       // LDS row pitch of one part, dwords (24 used)
static_assert((kWaves - 2) / kPairsPerRow + 1 + kK <= kRing, "rows of one step of 8 pairs");
static_assert(kWaves < kPairsPerRow, "at most one new row per step");
// a wave loads the weights of its next pair, kWaves pairs further on
constexpr int64_t kWeightBytes = (kPairs + kWaves) * kParts3 * kFc1PairBytes16;

// first pair of range s (whole groups of 4 pairs: 120 or 124 pairs each)
__host__ __device__ constexpr int range_begin(int s) { return 4 * (kPairs / 4 * s / kSplits); }

// The conv filters and biases in fp32, and the magnitude below which a pixel can
// be taken apart (see plain_patch).
struct ConvF32 {
  const float* w;
  const float* b;
  float limit;
};

// Block of 16 kTiles patches and 128 / kParts outputs.  LDS (dwords): ring
// [part][row][patch] | conv filters | row descriptors | per patch the 16-output
// tiles to compute in plain fp32, a bit each; the reduction reuses it up to the descriptors.
template <int kTiles, int kParts>
struct Block {
  static constexpr int kBt = 16 * kTiles;
  static constexpr int kMT = kMTiles / kParts;             // output tiles per wave
  static constexpr int kSlot = kBt * kRP;                  // dwords per row and part
  static constexpr int kPart = kRing * kSlot;
  static constexpr int kConvOff = kParts3 * kPart;
  // the reduction, at most 16 accumulator tiles a pass, of each one from each
  // of the other 7 waves
  static constexpr int kSlots = kMT * kTiles;
  static constexpr int kPer = kSlots >= kWaves ? kSlots / kWaves : 1;   // tiles a wave finishes
  static constexpr int kPass = kPer < 2 ? kPer : 2;        // of them per pass
  static constexpr int kOwners = kSlots / kPer;
  static constexpr int kRed = kOwners * kPass * (kWaves - 1) * 256;
  static constexpr int kConvEnd = kConvOff + kParts3 * 6 * 64 * 4;
  static constexpr int kDescOff = kConvEnd > kRed ? kConvEnd : kRed;
  static constexpr int kFlagOff = kDescOff + kBt * 4;
  static constexpr int kLds = kFlagOff + kBt;
  // register sets of weights: one wave's L2 latency is behind as many output tiles
  static constexpr int kSets = kTiles == 4 ? 3 : 6;
  static constexpr int kRowAll = kBt * kRowChunks;         // chunks per row
  static constexpr int kRowPer = (kRowAll + kThreads - 1) / kThreads;
  static_assert(kLds * 4 <= 160 * 1024 && kPer % kPass == 0 && kQ * kMT % kSets == 0 && kRowAll % 64 == 0, "block");
};

// a == high + middle + low exactly, and b, a's parts in the low halves: high is a
// rounded to bf16 (nearest even), middle the rest of at most 16 bits rounded, low
// the rest of at most 8.  (Below 2^-109 the low part is cut off under 2^-133.)
// Cut instead of rounded, the parts cost 1 % less time (event) and a product can
// be off by 2^-22.7.
__device__ __forceinline__ void split3(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  using Op = Op16<false>;
  h = Op::pack(a, b);
  a -= __uint_as_float(h << 16);
  b -= __uint_as_float(h & 0xFFFF0000u);
  m = Op::pack(a, b);
  a -= __uint_as_float(m << 16);
  b -= __uint_as_float(m & 0xFFFF0000u);
  l = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);   // the upper halves
}
__device__ __forceinline__ floatx4 mfma(const uint4& a, const uint4& b, const floatx4& c) {
  return Op16<false>::mfma(a, b, c);
}
// c += a x b, the smallest products first.  Two patch tiles take turns: an MFMA
// would wait a few cycles for an accumulator written by the one just before.
constexpr int kPartA[6] = {2, 0, 1, 1, 0, 0}, kPartB[6] = {0, 2, 1, 0, 1, 0};
__device__ __forceinline__ floatx4 mfma6(const uint4 (&a)[kParts3], const uint4 (&b)[kParts3], floatx4 c) {
#pragma unroll
  for (int k = 0; k < 6; ++k) c = mfma(a[kPartA[k]], b[kPartB[k]], c);
  return c;
}
__device__ __forceinline__ void mfma6x2(const uint4 (&a)[kParts3], const uint4 (&b0)[kParts3],
                                        const uint4 (&b1)[kParts3], floatx4& c0, floatx4& c1) {
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    c0 = mfma(a[kPartA[k]], b0[kPartB[k]], c0);
    c1 = mfma(a[kPartA[k]], b1[kPartB[k]], c1);
  }
}

// The FC1 sums of one patch (row descriptor d) over pairs P0 .. P_end - 1 in
// plain fp32, by the whole block, to dst[128] for the 16-output tiles of `tiles`.
// The window of a pair has six columns, the taps of the one that a position does
// not use are 0, as in the MFMA kernels: an infinite or NaN pixel makes the maps
// of both positions NaN, which the ReLU takes to 0.  0.15 ms a patch and
// block; LDS is free to use from the start.
constexpr int kPlainPairs = 4;                // pairs of a pass, one per 128 threads
constexpr int kPlainRows = 11;                // input rows of a range of at most 31 groups of 4 pairs
static_assert((4 * ((kPairs / 4 + kSplits - 1) / kSplits) - 1 + kPairsPerRow - 1) / kPairsPerRow + kK <= kPlainRows, "rows");
__device__ __forceinline__ void plain_patch(float* lds, const uint4& d, int P0, int P_end, uint32_t tiles,
                                            const uint4* __restrict__ w1p, const ConvF32& conv, float* dst) {
  typedef __attribute__((address_space(1))) const float* gptr;
  static_assert(kPlainPairs * 128 == kThreads && kPlainPairs * 2 * kCh <= kThreads, "threads of a pass");
  constexpr int kMaps = kPlainRows * kPatch, kSums = kMaps + kPlainPairs * 2 * kCh;
  const int tid = threadIdx.x, r0 = P0 / kPairsPerRow, rows = (P_end - 1) / kPairsPerRow + kK - r0;
  __syncthreads();
  for (int i = tid; i < rows * kPatch; i += kThreads) {
    const uint32_t r = (uint32_t)(r0 + i / kPatch), c = (uint32_t)(i % kPatch);
    const bool in = r >= (d.w & 255u) && r < ((d.w >> 8) & 255u) && c >= ((d.w >> 16) & 255u) && c < d.w >> 24;
    lds[i] = in ? ((gptr)row_chunk_addr(d, (int)r, 0))[c] : 0.f;
  }
  const int o = tid & 127, g = tid >> 7;
  const bool mine = (tiles >> (o / 16) & 1u) != 0;
  float acc = 0.f;
  for (int P = P0; P < P_end; P += kPlainPairs) {
    __syncthreads();
    if (tid < kPlainPairs * 2 * kCh) {
      const int ch = tid % kCh, s = tid / kCh % 2, Pm = P + tid / (2 * kCh);
      const float* x = lds + (Pm / kPairsPerRow - r0) * kPatch + 2 * (Pm % kPairsPerRow);
      float m = 0.f;
      for (int f = 0; f < 30; ++f) {
        const int u = f / 6, c = f % 6 - s;
        m = fmaf(c >= 0 && c < kK ? conv.w[ch * kK * kK + u * kK + c] : 0.f, x[u * kPatch + f % 6], m);
      }
      lds[kMaps + tid] = fmaxf(m + conv.b[ch], 0.f);
    }
    __syncthreads();
    if (mine) {
      // the weights from their parts (an exact sum), in the order of pack_fc1_f32_kernel
      float sum = 0.f;
      for (int k = 0; k < kQ * 4; ++k) {
        const int q = k >> 2, sub = k & 3;
        const uint4* w = w1p + (((int64_t)(P + g) * kQ + q) * kMTiles + o / 16) * kParts3 * 64 + 16 * sub + (o & 15);
        const uint4 part[kParts3] = {w[0], w[64], w[128]};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          float v[kParts3];
#pragma unroll
          for (int t = 0; t < kParts3; ++t) {
            const uint32_t dw = j < 2 ? part[t].x : j < 4 ? part[t].y : j < 6 ? part[t].z : part[t].w;
            v[t] = __uint_as_float(j & 1 ? dw & 0xFFFF0000u : dw << 16);
          }
          const int st = 2 * q + (j >> 2);
          sum = fmaf((v[0] + v[1]) + v[2],
                     lds[kMaps + g * 2 * kCh + st / 3 * kCh + 16 * (st % 3) + 4 * sub + (j & 3)], sum);
        }
      }
      acc += sum;
    }
  }
  __syncthreads();
  lds[kSums + tid] = acc;
  __syncthreads();
  if (tid < 128 && mine)
    dst[o] = (lds[kSums + tid] + lds[kSums + 128 + tid]) + (lds[kSums + 256 + tid] + lds[kSums + 384 + tid]);
}

// One block: patches p_base .. p_base + kBt - 1 (those past the batch hold
// zeros and are not stored), range `split`, output part `opart`.
template <int kTiles, int kParts>
__device__ __forceinline__ void conv_fc1_f32_block(uint32_t* lds, int split, int opart, int64_t p_base,
                                                   const HitSource& src, const uint4* __restrict__ w1p,
                                                   const uint4* __restrict__ convp, const ConvF32& conv,
                                                   float* __restrict__ part) {
  using B = Block<kTiles, kParts>;
  constexpr int kSlot = B::kSlot, kMT = B::kMT, kSets = B::kSets, kBt = B::kBt;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int P0 = range_begin(split), P_end = range_begin(split + 1);
  const int steps = (P_end - P0 + kWaves - 1) / kWaves;

  // FC1 fragments through a buffer resource (the pair after the last one is read
  // too, and allocated: the bounds check leaves out the scalar offset):
  // group G of a pair is K-step G / kMT, output tile G % kMT
  const __amdgpu_buffer_rsrc_t w1r = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint4*>(w1p), (short)0, (int)kWeightBytes, 0x00020000);
  const int voff = lane * 16 + opart * kMT * kParts3 * 1024;
  auto load_set = [&](int P, int G, uint4 (&w)[kParts3]) {
#pragma unroll
    for (int k = 0; k < kParts3; ++k)
      w[k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                           w1r, voff + k * 1024,
                                           ((P * kQ + G / kMT) * kMTiles + G % kMT) * kParts3 * 1024, 0));
  };
  uint4 w[kSets][kParts3];
#pragma unroll
  for (int s = 0; s < kSets; ++s) load_set(P0 + wave, s, w[s]);

  // ---- patch rows
  uint4* desc = reinterpret_cast<uint4*>(lds + B::kDescOff);
  uint32_t* flags = lds + B::kFlagOff;       // what to compute in plain fp32
  if (tid < kBt) {
    desc[tid] = src.get(p_base + tid);
    flags[tid] = 0;
  }
  uint4* filters = reinterpret_cast<uint4*>(lds + B::kConvOff);
  for (int i = tid; i < kParts3 * 6 * 64; i += kThreads) filters[i] = convp[i];
  __syncthreads();
  struct Row {
    rowx4 v[B::kRowPer];
    uint32_t kinds;
  };
  auto load_row = [&](int r, Row& row) {
    row.kinds = 0;
#pragma unroll
    for (int k = 0; k < B::kRowPer; ++k) {
      const int c = tid + k * kThreads;
      if (c < B::kRowAll) {
        uint32_t kind;
        row.v[k] = row_chunk_load(desc_from_lds(desc + c / kRowChunks), r, c - (c / kRowChunks) * kRowChunks,
                                  w1p, &kind);
        row.kinds |= kind << 2 * k;
      }
    }
  };
  auto store_row = [&](int r, const Row& row) {
#pragma unroll
    for (int k = 0; k < B::kRowPer; ++k) {
      const int c = tid + k * kThreads;
      if (c < B::kRowAll) {
        const int p = c / kRowChunks, h = c - (c / kRowChunks) * kRowChunks;
        const rowx4 x = row_chunk_finish(desc + p, r, h, row.v[k], (row.kinds >> 2 * k) & 3);
        bool fits = true;
#pragma unroll
        for (int j = 0; j < 4; ++j) fits &= fabsf(x[j]) < conv.limit;
        if (!fits) flags[p] = ~0u;
        uint2 hi, mi, lo;
        split3(x[0], x[1], hi.x, mi.x, lo.x);
        split3(x[2], x[3], hi.y, mi.y, lo.y);
        uint32_t* d = lds + r % kRing * kSlot + p * kRP + h * 2;
        *reinterpret_cast<uint2*>(d) = hi;
        *reinterpret_cast<uint2*>(d + B::kPart) = mi;
        *reinterpret_cast<uint2*>(d + 2 * B::kPart) = lo;
      }
    }
  };
  auto top_row = [&](int step) {             // highest input row a step needs
    const int pl = P0 + kWaves * step + kWaves - 1;
    return (pl < P_end ? pl : P_end - 1) / kPairsPerRow + kK - 1;
  };
  int loaded = top_row(0);
  {
    const int r0 = P0 / kPairsPerRow;
    Row row[kRing];
#pragma unroll
    for (int j = 0; j < kRing; ++j)
      if (r0 + j <= loaded) load_row(r0 + j, row[j]);
#pragma unroll
    for (int j = 0; j < kRing; ++j)
      if (r0 + j <= loaded) store_row(r0 + j, row[j]);
  }

  // this lane's 4 window dwords: slots f, f + 1 (f = 8 grp + 2d) are pixels
  // (u, c), (u, c + 1); kept as u | c / 2 << 4 in byte d (registers are what the
  // 64-patch loop is short of: three scratch loads a step fewer, event 6.11 -> 6.09 ms)
  uint32_t wpix = 0;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    int f = 8 * grp + 2 * d;
    if (f > 28) f = 28;                      // slots 30-31 are constants (set below)
    wpix |= (uint32_t)(f / 6 | (f % 6) / 2 << 4) << 8 * d;
  }
  const bool const_slot = grp == 3;

  // part k of the window of patch tile i at the lane's four places
  auto read_win = [&](const uint32_t (&base)[4], int i, int k) {
    const uint32_t* s = lds + k * B::kPart + i * 16 * kRP;
    uint4 win;
    win.x = s[base[0]];
    win.y = s[base[1]];
    win.z = s[base[2]];
    win.w = s[base[3]];
    asm volatile("" : "+v"(win.w));          // read by every lane: a select, not a branch
    win.w = const_slot ? (k == 0 ? 0x00003F80u : 0u) : win.w;
    return win;
  };
  // ReLU, and the maps of two conv tiles into an FC1 operand
  auto split_maps = [](const floatx4& ca, const floatx4& cb, uint4 (&b)[kParts3]) {
    split3(fmaxf(ca[0], 0.f), fmaxf(ca[1], 0.f), b[0].x, b[1].x, b[2].x);
    split3(fmaxf(ca[2], 0.f), fmaxf(ca[3], 0.f), b[0].y, b[1].y, b[2].y);
    split3(fmaxf(cb[0], 0.f), fmaxf(cb[1], 0.f), b[0].z, b[1].z, b[2].z);
    split3(fmaxf(cb[2], 0.f), fmaxf(cb[3], 0.f), b[0].w, b[1].w, b[2].w);
  };

  floatx4 acc[kMT][kTiles];
#pragma unroll
  for (int m = 0; m < kMT; ++m)
#pragma unroll
    for (int i = 0; i < kTiles; ++i) acc[m][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
  __syncthreads();                           // the first rows and the filters

#pragma unroll 1
  for (int step = 0; step < steps; ++step) {
    const int P = P0 + kWaves * step + wave;
    const bool new_row = step + 1 < steps && top_row(step + 1) > loaded;   // block-uniform
    Row row;
    if (P < P_end) {                         // (the last step of a range can be half a step)
      const int y = P / kPairsPerRow;
      const uint32_t at = (uint32_t)(y % kRing * kSlot), xh = (uint32_t)(P - y * kPairsPerRow);
      uint32_t base[4], wp = wpix;
      asm volatile("" : "+v"(wp));           // unpacked here, not once for the loop
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const uint32_t t = (wp >> 8 * d & 15u) * kSlot + at, c2 = wp >> (8 * d + 4) & 15u;
        base[d] = min(t, t - (uint32_t)(kRing * kSlot)) + (uint32_t)(col * kRP) + c2 + xh;   // wrapped
      }
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        // conv tiles (shift, channel tile) of K-step q, see conv_fc1_16.hip
        const int ta = (q == 2) ? 3 + 1 : (q == 1 ? 2 : 0), tb = (q == 0) ? 1 : (q == 1 ? 3 : 3 + 2);
        // The conv is a chain of LDS reads, MFMAs and conversions; a wave in it
        // goes first, and the other wave of the SIMD fills its gaps with FC1
        // (event: 6.18 -> 6.01 ms, with the two chains in turn 5.96)
        __builtin_amdgcn_s_setprio(2);
        uint4 b[kTiles][kParts3];
        if constexpr (kTiles < 4) {
          // with registers for it, the chains of all tiles and both conv tiles in
          // turn, then the conversions (235 patches 85.2 -> 83.4 us per call, 400 88.5
          // -> 86.3: an MFMA otherwise waits for the one before it)
          floatx4 ca[kTiles], cb[kTiles];
          uint4 win[kTiles][kParts3], fa[kParts3], fb[kParts3];
#pragma unroll
          for (int k = 0; k < kParts3; ++k) {
            fa[k] = filters[(k * 6 + ta) * 64 + lane];
            fb[k] = filters[(k * 6 + tb) * 64 + lane];
          }
#pragma unroll
          for (int i = 0; i < kTiles; ++i) {
#pragma unroll
            for (int k = 0; k < kParts3; ++k) win[i][k] = read_win(base, i, k);
            ca[i] = cb[i] = (floatx4){0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
          for (int k = 0; k < 6; ++k)
#pragma unroll
            for (int i = 0; i < kTiles; ++i) {
              ca[i] = mfma(fa[kPartA[k]], win[i][kPartB[k]], ca[i]);
              cb[i] = mfma(fb[kPartA[k]], win[i][kPartB[k]], cb[i]);
            }
#pragma unroll
          for (int i = 0; i < kTiles; ++i) split_maps(ca[i], cb[i], b[i]);
        } else {
#pragma unroll
          for (int i = 0; i < kTiles; ++i) {
            // (filter and window part by part: the window first, as above, made the
            // 64-patch loop wait more, event 6.11 -> 6.47 ms)
            uint4 win[kParts3], f[kParts3];
#pragma unroll
            for (int k = 0; k < kParts3; ++k) {
              f[k] = filters[(k * 6 + ta) * 64 + lane];
              win[k] = read_win(base, i, k);
            }
            const floatx4 z = {0.f, 0.f, 0.f, 0.f};
            const floatx4 ca = mfma6(f, win, z);
#pragma unroll
            for (int k = 0; k < kParts3; ++k) f[k] = filters[(k * 6 + tb) * 64 + lane];
            const floatx4 cb = mfma6(f, win, z);
            split_maps(ca, cb, b[i]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        // the next row's loads: behind this K-step's FC1
        if (q == kQ - 1 && new_row) load_row(loaded + 1, row);
#pragma unroll
        for (int m = 0; m < kMT; ++m) {
          constexpr int kAll = kQ * kMT;
          const int G = q * kMT + m, s = G % kSets;
#pragma unroll
          for (int i = 0; i + 1 < kTiles; i += 2) mfma6x2(w[s], b[i], b[i + 1], acc[m][i], acc[m][i + 1]);
          if constexpr (kTiles == 1) acc[m][0] = mfma6(w[s], b[0], acc[m][0]);
          load_set(G + kSets < kAll ? P : P + kWaves, (G + kSets) % kAll, w[s]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (new_row) {
      // the slot that the row takes held a row of this step
      __syncthreads();
      store_row(++loaded, row);
      __syncthreads();
    }
  }

  // ---- fixed-order sum over the waves, each finishing its share of the tiles:
  //      ((g0 + g4) + (g1 + g5)) + ((g2 + g6) + (g3 + g7))
  constexpr int kPer = B::kPer, kPass = B::kPass, kOwners = B::kOwners;
  constexpr int kStride = kWaves / kOwners;                // owner o is wave o * kStride
  floatx4* red = reinterpret_cast<floatx4*>(lds);
  float* dst = part + ((int64_t)split * src.n + p_base) * kFc1Out;
  auto entry = [&](int o, int j, int from) { return ((o * kPass + j) * (kWaves - 1) + from) * 64 + lane; };
#pragma unroll
  for (int j0 = 0; j0 < kPer; j0 += kPass) {
    __syncthreads();                         // the ring, or the last pass, is dead
#pragma unroll
    for (int k = 0; k < kOwners * kPass; ++k) {
      const int o = k / kPass, j = k % kPass, q = o * kPer + j0 + j, g = o * kStride;
      if (wave != g) red[entry(o, j, wave - (wave > g ? 1 : 0))] = acc[q / kTiles][q % kTiles];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kOwners * kPass; ++k) {
      const int o = k / kPass, j = k % kPass, q = o * kPer + j0 + j, g0 = o * kStride;
      if (wave == g0) {
        floatx4 v[kWaves];
#pragma unroll
        for (int g = 0; g < kWaves; ++g)
          v[g] = g == g0 ? acc[q / kTiles][q % kTiles] : red[entry(o, j, g - (g > g0 ? 1 : 0))];
        const floatx4 sum = ((v[0] + v[4]) + (v[1] + v[5])) + ((v[2] + v[6]) + (v[3] + v[7]));
        const int p = 16 * (q % kTiles) + col, out = 16 * (opart * kMT + q / kTiles) + 4 * grp;
        const floatx4 z = sum * 0.f;
        if (!((z[0] + z[1]) + (z[2] + z[3]) == 0.f)) atomicOr(&flags[p], 1u << out / 16);   // not finite
        if (p_base + p < src.n) __builtin_nontemporal_store(sum, reinterpret_cast<floatx4*>(dst + p * kFc1Out + out));
      }
    }
  }

  // ---- the patches without a place in three parts, one after the other (the
  // stores above to their sums come before the barrier, these after it)
  __syncthreads();
  uint64_t todo = __ballot(lane < kBt && flags[lane < kBt ? lane : 0] != 0 && p_base + lane < src.n);
  while (todo) {                             // the same in every wave
    const int p = __ffsll((unsigned long long)todo) - 1;
    todo &= todo - 1;
    plain_patch(reinterpret_cast<float*>(lds), desc_from_lds(desc + p), P0, P_end,
                flags[p] & ((1u << kMT) - 1) << opart * kMT, w1p, conv, dst + p * kFc1Out);
  }
}

// Tiles t < n_big hold 64 patches, the ones after them 32.  Block b runs on XCD
// b % 8, whose L2 the blocks there share for their range's weights; the ranges
// move on by one XCD every round of the CUs (a row of the grid), because two of
// the eight are 3 % longer.  256 registers, 51 more spilled: nearly all of them
// around the first rows; the 64-patch loop holds 9 scratch loads and 6 stores
// per 720 MFMAs.
__global__ __launch_bounds__(kThreads, 1) void conv_fc1_f32_kernel(HitSource src, int64_t n_big,
                                                                   const uint4* __restrict__ w1p,
                                                                   const uint4* __restrict__ convp, ConvF32 conv,
                                                                   float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) uint32_t lds[Block<4, 1>::kLds];
  const int64_t t = blockIdx.y * (gridDim.x / kSplits) + blockIdx.x / kSplits;
  const int split = (int)((blockIdx.x + blockIdx.y) % kSplits);
  const int64_t p_base = t < n_big ? t * 64 : n_big * 64 + (t - n_big) * 32;
  if (p_base >= src.n) return;               // (the last row)
  if (t < n_big)
    conv_fc1_f32_block<4, 1>(lds, split, 0, p_base, src, w1p, convp, conv, part);
  else
    conv_fc1_f32_block<2, 1>(lds, split, 0, p_base, src, w1p, convp, conv, part);
}

// Block b: split b % kSplits, then output part, then patch tile.
template <int kTiles, int kParts>
__global__ __launch_bounds__(kThreads, 1) void conv_fc1_f32_small_kernel(HitSource src,
                                                                         const uint4* __restrict__ w1p,
                                                                         const uint4* __restrict__ convp, ConvF32 conv,
                                                                         float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) uint32_t lds[Block<kTiles, kParts>::kLds];
  const int split = blockIdx.x % kSplits;
  const int64_t r = blockIdx.x / kSplits;
  conv_fc1_f32_block<kTiles, kParts>(lds, split, (int)(r % kParts), r / kParts * (16 * kTiles), src, w1p, convp,
                                     conv, part);
}

// The parts of a weight: rounded to nearest (their products' rest is then of
// either sign), cut where that would round a finite weight to infinity.
__device__ __forceinline__ void round3(float v, float (&out)[kParts3]) {
#pragma unroll
  for (int k = 0; k < kParts3; ++k) {
    float h = Op16<false>::value((uint16_t)Op16<false>::pack(v, 0.f));
    if (isinf(h)) h = __uint_as_float(__float_as_uint(v) & 0xFFFF0000u);
    out[k] = h;
    v = isfinite(v) ? v - h : 0.f;
  }
}
__device__ __forceinline__ void store3(const float (&v)[8], uint4* out, int stride) {
  float p[8][kParts3];
#pragma unroll
  for (int j = 0; j < 8; ++j) round3(v[j], p[j]);
  using Op = Op16<false>;
#pragma unroll
  for (int k = 0; k < kParts3; ++k)          // (every part is a bf16 value: packing is exact)
    out[k * stride] = make_uint4(Op::pack(p[0][k], p[1][k]), Op::pack(p[2][k], p[3][k]),
                                 Op::pack(p[4][k], p[5][k]), Op::pack(p[6][k], p[7][k]));
}

// FC1 weights in the order the kernel reads them, once at create: one thread
// per (pair, K-step, 16 outputs, lane (output i, K-slot group g)).
__global__ __launch_bounds__(256) void pack_fc1_f32_kernel(const float* __restrict__ w1, uint4* __restrict__ out) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= kFc1Frags) return;
  const int lane = (int)(idx & 63);
  const int64_t f = idx >> 6;
  const int m = (int)(f % kMTiles), q = (int)(f / kMTiles % kQ);
  const int64_t P = f / (kMTiles * kQ);
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int st = 2 * q + (j >> 2);         // conv tile: shift st / 3, channel tile st % 3
    const int64_t k = (2 * P + st / 3) * kCh + 16 * (st % 3) + 4 * (lane >> 4) + (j & 3);
    v[j] = w1[k * kFc1Out + 16 * m + (lane & 15)];
  }
  store3(v, out + f * kParts3 * 64 + lane, 64);
}

// The conv filters [part][shift][channel tile][64 lanes], slot 30 the bias.
__global__ __launch_bounds__(64) void pack_conv_f32_kernel(const float* __restrict__ K, const float* __restrict__ b,
                                                           uint4* __restrict__ out) {
  const int st = blockIdx.x, s = st / 3, lane = threadIdx.x;
  const int ch = 16 * (st % 3) + (lane & 15);
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int f = 8 * (lane >> 4) + j, u = f / 6, c = f % 6 - s;
    v[j] = f == 30 ? b[ch] : (f < 30 && c >= 0 && c < kK) ? K[ch * kK * kK + u * kK + c] : 0.f;
  }
  store3(v, out + st * 64 + lane, 6 * 64);
}

}  // namespace

int conv_fc1_f32_splits() { return kSplits; }
// Pixels below the limit keep every sum of products of a conv, in whatever order
// and by parts, below a quarter of fp32's range (parts may be of either sign and
// add up to 1.02 times their value).  0, which no pixel is below, where a filter or
// a bias leaves no room or is not finite itself.
float conv_fc1_f32_limit(const float* conv_w, const float* conv_b) {
  constexpr double kRoom = 0x1p126;
  double limit = kRoom;
  for (int k = 0; k < kCh; ++k) {
    double sum = 0.0;
    for (int i = 0; i < kK * kK; ++i) sum += std::fabs((double)conv_w[k * kK * kK + i]);
    const double at = (kRoom - 1.02 * std::fabs((double)conv_b[k])) / std::max(1.02 * sum, 1.0);
    limit = at < limit ? at : limit;
    if (!(at > 0)) return 0.f;
  }
  return (float)limit;
}
int64_t conv_fc1_f32_weight_bytes() { return kWeightBytes; }

// Tiles that one round of the CUs holds.
static int64_t tiles_per_round(int cus) { return cus >= kSplits ? cus / kSplits : 1; }

// Small batches: patches per block and output parts, (0, 0) past 512 patches
// on 256 CUs.  The shapes whose blocks fit one round of the CUs, by the time of
// a K-step in the block (two waves per SIMD, 16 cycles per MFMA; 3 KiB of
// weights per wave and output tile at 64 B per clock and CU, whichever is
// longer): 16 patches, a quarter of the outputs 770 cycles; 32 patches, a
// quarter 1,540, half 2,300; 32 patches and all outputs 3,840 (the blocks of
// the other kernel).
void conv_fc1_f32_small(int64_t n, int cus, int* tiles, int* parts) {
  const int64_t per_round = tiles_per_round(cus);
  *tiles = *parts = 0;
  if ((n + 15) / 16 * 4 <= per_round) {
    *tiles = 1;
    *parts = 4;
  } else if ((n + 31) / 32 * 4 <= per_round) {
    *tiles = 2;
    *parts = 4;
  } else if ((n + 31) / 32 * 2 <= per_round) {
    *tiles = 2;
    *parts = 2;
  }
}

// Tiles of 64 patches fill whole rounds of the CUs (one block per CU); the
// rest is cut into tiles of 32 when those fit in one round, which then takes
// about half as long.
void conv_fc1_f32_tiles(int64_t n, int cus, int64_t* n_big, int64_t* n_small) {
  const int64_t per_round = tiles_per_round(cus);
  int64_t big = n / (64 * per_round) * per_round;
  const int64_t rest = n - big * 64;
  int64_t small = (rest + 31) / 32;
  if (small > per_round) {
    big += (rest + 63) / 64;
    small = 0;
  }
  *n_big = big;
  *n_small = small;
}

hipError_t launch_pack_f32(const float* conv_w, const float* conv_b, const float* fc1_w, uint4* conv_frag,
                           uint4* fc1_frag, hipStream_t stream) {
  const hipError_t e = launch_kernel(pack_conv_f32_kernel, dim3(6), dim3(64), 0, stream, conv_w, conv_b, conv_frag);
  if (e != hipSuccess) return e;
  return launch_kernel(pack_fc1_f32_kernel, dim3((unsigned)((kFc1Frags + 255) / 256)), dim3(256), 0, stream, fc1_w,
                       fc1_frag);
}

hipError_t launch_conv_fc1_f32(const RowInput& in, int64_t n, const DeviceWeights& w, float* part, int cus,
                               hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const uint4 *w1p = w.fc1_frag, *convp = w.conv_frag;
  const ConvF32 conv = {w.conv_w, w.conv_b, w.conv_limit};
  const HitSource src = hit_source(in, n);
  int tiles = 0, parts = 0;
  conv_fc1_f32_small(n, cus, &tiles, &parts);
  if (tiles) {
    const dim3 grid((unsigned)((n + 16 * tiles - 1) / (16 * tiles) * parts * kSplits));
    auto go = [&](auto kernel) { return launch_kernel(kernel, grid, dim3(kThreads), 0, stream, src, w1p, convp, conv, part); };
    if (tiles == 1) return go(conv_fc1_f32_small_kernel<1, 4>);
    return parts == 4 ? go(conv_fc1_f32_small_kernel<2, 4>) : go(conv_fc1_f32_small_kernel<2, 2>);
  }
  int64_t n_big = 0, n_small = 0;
  conv_fc1_f32_tiles(n, cus, &n_big, &n_small);
  const int64_t round = tiles_per_round(cus), all = n_big + n_small;
  const dim3 grid((unsigned)((all < round ? all : round) * kSplits), (unsigned)((all + round - 1) / round));
  return launch_kernel(conv_fc1_f32_kernel, grid, dim3(kThreads), 0, stream, src, n_big, w1p, convp, conv, part);
}

}  // namespace pointid
