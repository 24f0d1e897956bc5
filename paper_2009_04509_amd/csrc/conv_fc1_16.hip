// Fused conv 5x5 (1->48) + ReLU + FC1 (92928->128) on 16-bit MFMA (paper §2.2),
// with bf16 or fp16 operands and fp32 accumulation.
//
// FC1 is a skinny, very deep GEMM (M = patches, N = 128, K = 92,928) whose A
// operand — the conv maps, 185,856 B per patch in 16 bits — would cost twice its
// size in HBM traffic if written out and read back.  Here the conv is FC1's
// operand producer: the maps exist only in registers.
//
// Work split.  A block owns 96 patches (64 in the blocks of the last rounds of
// some batches: see conv_fc1_16_tiles; small batches run the thin tiles
// further below, with the same sums) and one of kSplits16 contiguous ranges of
// map positions (split-K), or 2 or 4 consecutive ones one after the other in
// batches of whole rounds of such blocks; blockIdx % 8 selects the range, so the
// blocks that run on one XCD stream the same weights (2.97 MB per range)
// through its 4 MB L2 at the same time.  Positions are taken in pairs (x, x+1) with x even: the
// 5x6 pixel window of a pair (30 values) fits one K=32 MFMA operand, shared by
// both positions.  The block's 8 waves (2 per SIMD, so one wave's conversions
// overlap the other's MFMAs) form 4 position groups x 2 output halves.  The two
// waves of a group take the same interleaved pairs; each computes the conv of
// half of the 96 patches, and the pair swaps the converted 16-bit fragments
// through LDS (double-buffered, one block barrier per K-step), so the conv is
// computed once and each wave streams only the FC1 weights of its 64 outputs:
// every weight fragment fetched through L1 feeds 6 MFMAs.  LDS also holds a
// ring of 8 patch rows (the 5 rows a map row needs, plus those prefetched two
// steps ahead) for the block's 96 patches, and the conv filter fragments.
//
// Per pair and per 16-patch tile, v_mfma_f32_16x16x32_{bf16,f16}:
//   conv:  D[ch][patch] = sum_slot Kc[ch][slot] * Win[slot][patch]
//          slot f < 30 holds window pixel (u, c) = (f / 6, f % 6), rows y+u and
//          columns x+c; the filter fragment for position x+s holds K[ch][u][c-s].
//          Slots 30 and 31 hold 1.0 in the window and the conv bias split into
//          two 16-bit halves (hi + lo) in the filter, so the fp32 accumulator
//          adds the bias at about twice the operand precision.
//   ReLU + round to 16 bits (RNE) on the accumulator lanes, then the 16x16 result
//   tile is used directly as the B operand of FC1: a lane holds output rows
//   4g..4g+3 for one patch column, which is the B operand's K-slot group g.  Two
//   conv tiles make one K=32 FC1 step; the FC1 weights are repacked at create
//   time into the matching K order, one 1 KiB fragment per (pair, step, 16 outputs).
//   FC1:   acc[n][patch] += W1t[n][k] * maps[k][patch]
//
// The four position groups' partial sums are added in LDS in a fixed order and
// written as fp32 partials [split][patch][128]; the tail kernel adds the splits.
#include <type_traits>

#include "internal.h"
#include "op16.h"
#include "rows.h"
#include "thin.h"

namespace pointid {
namespace {

constexpr int kSplits16 = 8;                  // position ranges (split-K), one per XCD
constexpr int kRing = 8;                      // patch-row ring slots
// rows the first steps of a range need: their pairs span at most two map rows,
// plus the filter height
constexpr int kPrologueRows = 2 + 5 - 1;
constexpr int kBigTile = 96;                  // patches per block (most blocks)
constexpr int kMidTile = 64;                  // patches per block (the last rounds, some batches)
// a wave loads the weights of its next pair, kKGroups pairs further on
constexpr int64_t kWeightBytes = (kPos / 2 + kKGroups) * kFc1PairBytes16;
static_assert(kFc1PairBytes16 * (kPos / 2) == kFc1Frags * 16, "packed pairs");

// First step (kKGroups pairs) of position range s, of 242 in all.
__host__ __device__ constexpr int range_begin(int s) {
  return (kPos / 2 / kKGroups) * s / kSplits16;
}

// Layout of a block of kBt patches.  LDS (dwords): ring | conv filter
// fragments | swap buffers; the reduction uses the swap buffers and the LDS
// behind them.
template <int kBt>
struct Tile {
  static constexpr int kTiles = kBt / 16;                 // 16-patch MFMA tiles
  static constexpr int kOwn = kTiles / kNHalves;          // tiles whose conv a wave computes
  static constexpr int kSlot = kBt * kRP;                 // dwords per ring slot
  static constexpr int kConvOff = kRing * kSlot;
  static constexpr int kSwapOff = kConvOff + 6 * 64 * 4;
  static constexpr int kSwapWave = kOwn * 64 * 4;         // one wave's fragments
  static constexpr int kSwapBuf = kWaves * kSwapWave;     // one buffer
  // the reduction: kRedTiles accumulator tiles per position group and pass, of
  // each one from each of the other three groups, per output half
  static constexpr int kRedTiles = kMT * kTiles / kKGroups / 2;
  static constexpr int kRed = kNHalves * kKGroups * kRedTiles * (kKGroups - 1) * 64 * 4;
  static constexpr int kLdsDwords = kSwapOff + (2 * kSwapBuf > kRed ? 2 * kSwapBuf : kRed);
  static_assert(kLdsDwords >= 2 * kRed, "one pass");
  static_assert(kTiles % kNHalves == 0 && kOwn <= 3, "whole tiles per output half");
};
static_assert(Tile<kBigTile>::kLdsDwords >= Tile<kMidTile>::kLdsDwords, "LDS sized by the big tile");
static_assert(Tile<kBigTile>::kLdsDwords * 4 <= 160 * 1024, "LDS of one block");

// A patch row of each of a block's kBt patches, in chunks of 16 bytes of `In`
// (16-bit patches from the gather, or fp32 pre-cut patches): chunk
// c = tid + k * kThreads, the last k for the first threads only (whole waves,
// so no lane diverges).  Patches past the end of the batch are read from the
// last patch instead: their results are never stored.  fp32 pixels stay as
// they are in registers and are rounded (nearest even) on their way into LDS,
// so that nothing waits for their loads in between.  (Rounding them in the
// kernel saves a pass that writes 16-bit patches: 31 of 429 us at 16,384
// patches.  Reading the rows of hits from the plane images here, without the
// gather's pass, gained nothing over an event: the conv's share of the power
// limit went to eight times the image reads.)
template <int kBt, class In>
struct Rows {
  static constexpr int kPix = 16 / (int)sizeof(In);
  static constexpr int kPerRow = kPatch / kPix;
  static constexpr int kAll = kBt * kPerRow;
  static constexpr int kPer = (kAll + kThreads - 1) / kThreads;      // chunks per thread
  static_assert(kAll % 64 == 0, "row chunks in whole waves");
  uint4 v[kPer];

  // streamed once per block: non-temporal, so the rows do not push the FC1
  // weights out of L2
  __device__ __forceinline__ void load(const In* __restrict__ patches, int64_t n, int64_t p_base, int r) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int c = threadIdx.x + k * kThreads;
      if (c < kAll) {
        const int p = c / kPerRow, h = c - (c / kPerRow) * kPerRow;
        int64_t gp = p_base + p;
        gp = gp < n ? gp : n - 1;
        const In* src = patches + gp * kPatchPix + r * kPatch + h * kPix;
        v[k] = __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src)));
      }
    }
  }
  template <bool kFp16>
  __device__ __forceinline__ void store(uint32_t* lds, int r) const {
    using Op = Op16<kFp16>;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int c = threadIdx.x + k * kThreads;
      if (c < kAll) {
        const int p = c / kPerRow, h = c - (c / kPerRow) * kPerRow;
        uint32_t* d = lds + (r & (kRing - 1)) * Tile<kBt>::kSlot + p * kRP + h * (kPix / 2);
        if constexpr (sizeof(In) == 2) {
          *reinterpret_cast<uint2*>(d) = make_uint2(v[k].x, v[k].y);
          *reinterpret_cast<uint2*>(d + 2) = make_uint2(v[k].z, v[k].w);
        } else {
          *reinterpret_cast<uint2*>(d) =
              make_uint2(Op::pack(__uint_as_float(v[k].x), __uint_as_float(v[k].y)),
                         Op::pack(__uint_as_float(v[k].z), __uint_as_float(v[k].w)));
        }
      }
    }
  }
};

// The rows of hits, read from the plane images (rows.h) with the descriptors at
// `desc` in LDS; patches past the end of the batch hold zeros.
template <int kBt>
struct Rows<kBt, HitSource> {
  static constexpr int kAll = kBt * kRowChunks;
  static constexpr int kPer = (kAll + kThreads - 1) / kThreads;
  static_assert(kAll % 64 == 0, "row chunks in whole waves");
  rowx4 v[kPer];
  uint32_t kinds;

  __device__ __forceinline__ void load(const uint4* desc, const void* safe, int r) {
    kinds = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int c = threadIdx.x + k * kThreads;
      if (c < kAll) {
        uint32_t kind;
        v[k] = row_chunk_load(desc_from_lds(desc + c / kRowChunks), r, c - (c / kRowChunks) * kRowChunks, safe, &kind);
        kinds |= kind << 2 * k;
      }
    }
  }
  template <bool kFp16>
  __device__ __forceinline__ void store(uint32_t* lds, const uint4* desc, int r) const {
    using Op = Op16<kFp16>;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int c = threadIdx.x + k * kThreads;
      if (c < kAll) {
        const int p = c / kRowChunks, h = c - (c / kRowChunks) * kRowChunks;
        const rowx4 x = row_chunk_finish(desc + p, r, h, v[k], (kinds >> 2 * k) & 3);
        *reinterpret_cast<uint2*>(lds + (r & (kRing - 1)) * Tile<kBt>::kSlot + p * kRP + h * 2) =
            make_uint2(Op::pack(x[0], x[1]), Op::pack(x[2], x[3]));
      }
    }
  }
};

// One block: patches p_base .. p_base + kBt - 1 (clamped to the batch) and
// `ranges` consecutive position ranges from `split0`.  The pairs of a range
// follow those of the range before it, so the patch rows in the ring run on
// over their boundary.  (kMulti: more than one; a kernel of its own for one,
// because the loop around the ranges costs registers and a pass.)
template <bool kFp16, int kBt, class In, bool kMulti>
__device__ __forceinline__ void conv_fc1_block(
    uint32_t* lds, int split0, int ranges_, int64_t p_base, const In* __restrict__ patches, int64_t n,
    const uint4* __restrict__ w1p, const uint4* __restrict__ convp, float* __restrict__ part) {
  using T = Tile<kBt>;
  constexpr bool kHits = std::is_same<In, HitSource>::value;
  uint4* desc = reinterpret_cast<uint4*>(lds + T::kLdsDwords);   // (hits only)
  if constexpr (kHits) {
    if (threadIdx.x < kBt) desc[threadIdx.x] = patches->get(p_base + threadIdx.x);
    __syncthreads();
  }
  auto load_row = [&](Rows<kBt, In>& row, int rr) {
    if constexpr (kHits) row.load(desc, w1p, rr);
    else row.load(patches, n, p_base, rr);
  };
  auto store_row = [&](const Rows<kBt, In>& row, int rr) {
    if constexpr (kHits) row.template store<kFp16>(lds, desc, rr);
    else row.template store<kFp16>(lds, rr);
  };
  const int ranges = kMulti ? ranges_ : 1;
  constexpr int kTiles = T::kTiles, kOwn = T::kOwn, kSlot = T::kSlot;
  constexpr int kSlots = kMT * kTiles;       // accumulator tiles of a wave
  constexpr int kPer = kSlots / kKGroups;    // tiles a wave finishes
  static_assert(kSlots % kKGroups == 0, "whole quarters");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave % kKGroups;            // position group
  const int nh = wave / kKGroups;            // output half; also the half of the tiles it convolves
  const int partner = kg + kKGroups * (1 - nh);
  const int col = lane & 15;                 // MFMA column (patch within tile) / row
  const int grp = lane >> 4;                 // MFMA K-slot group
  // range boundaries on whole steps of kKGroups pairs: every wave runs as many pairs
  const int P0 = kKGroups * range_begin(split0);
  const int P_last = kKGroups * range_begin(split0 + ranges) - 1;
  using Op = Op16<kFp16>;

  // conv filter fragments [shift][channel tile] in LDS; a K-step reads two
  // (copied below, with the first patch rows, so both loads are in flight together)
  uint4* cwl = reinterpret_cast<uint4*>(lds + T::kConvOff);
  static_assert(6 * 64 <= kThreads, "one filter chunk per thread");
  // swap buffers: [buffer][wave][own tile][lane] x 16 B
  uint4* swp = reinterpret_cast<uint4*>(lds + T::kSwapOff);

  // this lane's 4 window dwords: slot pair f = 8*grp + 2d -> pixel (u, c), kept
  // as u | c / 2 << 4 in byte d (registers are what bounds this kernel)
  uint32_t wpix = 0;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    int f = 8 * grp + 2 * d;
    if (f > 28) f = 28;                      // slots 30-31 are constants (masked below)
    wpix |= (uint32_t)((f / 6) | (f % 6) / 2 << 4) << (8 * d);
  }
  const int wcol = col * kRP + nh * kOwn * 16 * kRP;
  const bool const_slot = (grp == 3);

  // ---- patch rows.  The window of step s+1 is read during step s.  Gathered and
  // pre-cut rows: a row's loads are issued at the start of a step and it goes
  // into the ring at its end, two steps ahead of the step that needs it, so that
  // no row is held in registers from one step to the next (2,600 pre-cut patches
  // 83.8 -> 79.1 us per call, 16,384 414.2 -> 401.3: fp32 rows spilled registers).
  // Rows of hits come from further away: they go into the ring a step after
  // their loads, three steps ahead (1,100 hits 59.2 us without, 58.2 with).
  constexpr bool kLate = kHits;
  constexpr int kAhead = kLate ? 3 : 2;
  static_assert(kKGroups * kAhead + kKGroups - 1 < kPairsPerRow && 1 + kK < kRing,
                "rows up to 1 + 4 past a step's first");
  auto top_row = [&](int step) {             // highest input row a step needs
    int pl = P0 + kKGroups * step + kKGroups - 1;
    if (pl > P_last) pl = P_last;
    return pl / kPairsPerRow + kK - 1;
  };
  // all rows in flight at once (at most kPrologueRows), then into the ring
  int loaded_hi = top_row(kAhead - 1);
  {
    const int r0 = P0 / kPairsPerRow;
    Rows<kBt, In> v[kPrologueRows];
    uint4 fv;
    if (tid < 6 * 64) fv = convp[tid];
#pragma unroll
    for (int j = 0; j < kPrologueRows; ++j)
      if (r0 + j <= loaded_hi) load_row(v[j], r0 + j);
    if (tid < 6 * 64) cwl[tid] = fv;
#pragma unroll
    for (int j = 0; j < kPrologueRows; ++j)
      if (r0 + j <= loaded_hi) store_row(v[j], r0 + j);
  }
  __syncthreads();

  // window of pair P; the constant slots are set by fix_win, which the main
  // loop issues a few MFMAs later so that no VALU op waits on the LDS reads
  auto read_win_raw = [&](int P, uint4 (&win)[kOwn]) {
    const int y = P / kPairsPerRow;
    const int xh = P - y * kPairsPerRow;     // x / 2
    int base[4];
    uint32_t wp = wpix;
    asm volatile("" : "+v"(wp));            // unpacked here, not once for the loop
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int u = (wp >> (8 * d)) & 15, c2 = (wp >> (8 * d + 4)) & 15;
      base[d] = ((y + u) & (kRing - 1)) * kSlot + wcol + c2 + xh;
    }
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      const int o = i * 16 * kRP;
      win[i].x = lds[base[0] + o];
      win[i].y = lds[base[1] + o];
      win[i].z = lds[base[2] + o];
      win[i].w = lds[base[3] + o];
    }
  };
  auto fix_win = [&](uint4 (&win)[kOwn]) {
#pragma unroll
    for (int i = 0; i < kOwn; ++i) win[i].w = const_slot ? Op::kOnes : win[i].w;
  };
  // filter fragments of K-step q: conv tiles (shift, channel tile) feeding it
  auto read_filters = [&](int q, uint4& fa, uint4& fb) {
    const int sa = (q == 2) ? 1 : 0, ta = (q == 0) ? 0 : (q == 1 ? 2 : 1);
    const int sb = (q == 0) ? 0 : 1, tb = (q == 0) ? 1 : (q == 1 ? 0 : 2);
    fa = cwl[(sa * 3 + ta) * 64 + lane];
    fb = cwl[(sb * 3 + tb) * 64 + lane];
  };
  // ReLU + round to 16 bits: a conv tile pair becomes an FC1 B operand
  auto convert1 = [&](const floatx4& ca, const floatx4& cb) {
    return make_uint4(relu2(Op::pack(ca[0], ca[1])), relu2(Op::pack(ca[2], ca[3])),
                      relu2(Op::pack(cb[0], cb[1])), relu2(Op::pack(cb[2], cb[3])));
  };
  auto put1 = [&](int buf, int i, const uint4& bf) {
    swp[((buf * kWaves + wave) * kOwn + i) * 64 + lane] = bf;
  };
  auto get_swap = [&](int buf, uint4 (&bf)[kOwn]) {
#pragma unroll
    for (int i = 0; i < kOwn; ++i) bf[i] = swp[((buf * kWaves + partner) * kOwn + i) * 64 + lane];
  };

  // FC1 fragments of this wave's outputs through a buffer resource: the
  // fragment's place is a scalar offset and the output tile an immediate one, so
  // the loads need one per-lane register, no per-lane arithmetic and one scalar
  // addition per K-step.  (The resource's bounds check does not cover the scalar
  // offset: the pair after a wave's last one is read, and allocated.)
  const __amdgpu_buffer_rsrc_t w1r = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint4*>(w1p), (short)0, (int)kWeightBytes, 0x00020000);
  const int voff = lane * 16 + nh * kMT * 1024;
  auto load_one = [&](int P, int q, int m) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                         w1r, voff + m * 1024, (P * 3 + q) * 8 * 1024, 0));
  };

  int step = 0;                              // of the block's first range on
  bool row_pending = false;                  // row loaded_hi + 1 is on its way, in rv
  Rows<kBt, In> rv;
#pragma unroll
  for (int k = 0; k < Rows<kBt, In>::kPer; ++k) rv.v[k] = {};
#pragma unroll 1
  for (int split = split0; split < split0 + ranges; ++split) {
  const int step_end = range_begin(split + 1) - range_begin(split0);
  // accumulators for the wave's own conv tiles (block tiles nh*kOwn + i) and
  // for the partner's (tiles (1-nh)*kOwn + i); indexed statically only, so
  // they stay in registers
  floatx4 acc_own[kMT][kOwn], acc_oth[kMT][kOwn];
#pragma unroll
  for (int m = 0; m < kMT; ++m)
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      acc_own[m][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
      acc_oth[m][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
    }

  // ---- software pipeline.  Entering a K-step, this wave's own conv fragments
  // are in registers and the partner's are in swap buffer `buf` (published by
  // the last barrier).  While the FC1 MFMAs run, the conv of the next K-step is
  // issued, converted and published in the other buffer.  The FC1 weights sit
  // in 3 register sets, one per K-step of a pair (set q for K-step q), each
  // fragment reloaded for the next pair as soon as its MFMAs have issued, two
  // and a half K-steps before it is used.
  uint4 w[3][kMT], win[kOwn], own[kOwn];
  {
    const int P = P0 + kKGroups * step + kg;
#pragma unroll
    for (int i = 0; i < 3 * kMT; ++i)        // in the loop's order, for exact wait counts
      w[i / kMT][i % kMT] = load_one(P, i / kMT, i % kMT);
    read_win_raw(P, win);
    fix_win(win);
    uint4 fa, fb;
    read_filters(0, fa, fb);
    const floatx4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kOwn; ++i) own[i] = convert1(Op::mfma(fa, win[i], z), Op::mfma(fb, win[i], z));
  }
  int buf = 0;
#pragma unroll
  for (int i = 0; i < kOwn; ++i) put1(buf, i, own[i]);
  __syncthreads();

#pragma unroll 1
  for (; step < step_end; ++step) {
    const int P = P0 + kKGroups * step + kg;
    uint4 win_next[kOwn];
    if constexpr (!kLate) {                  // block-uniform
      row_pending = top_row(step + kAhead) > loaded_hi;
      if (row_pending) load_row(rv, loaded_hi + 1);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int nq = (q + 1) % 3;            // the next K-step
      uint4 oth[kOwn], nxt[kOwn], fa, fb;
      floatx4 ca[kOwn], cb[kOwn];
      const floatx4 z = {0.f, 0.f, 0.f, 0.f};
      // One K-step in ten groups of 3 MFMAs, the other work spread between
      // them: the two waves sharing a SIMD run the same sequence at about the
      // same time, so neither may bunch its VALU or LDS work.
      auto own_group = [&](int m) {
#pragma unroll
        for (int i = 0; i < kOwn; ++i) acc_own[m][i] = Op::mfma(w[q][m], own[i], acc_own[m][i]);
      };
      auto oth_group = [&](int m) {
#pragma unroll
        for (int i = 0; i < kOwn; ++i) acc_oth[m][i] = Op::mfma(w[q][m], oth[i], acc_oth[m][i]);
      };
      // g0: next filters, then the partner's fragments, from LDS (LDS returns
      // in order, and the filters are needed first)
      read_filters(nq, fa, fb);
      get_swap(buf, oth);
      own_group(0);
      __builtin_amdgcn_sched_barrier(0);
      own_group(1);
      __builtin_amdgcn_sched_barrier(0);
      // g2, g3: conv of the next K-step
#pragma unroll
      for (int i = 0; i < kOwn; ++i) ca[i] = Op::mfma(fa, (q == 2) ? win_next[i] : win[i], z);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kOwn; ++i) cb[i] = Op::mfma(fb, (q == 2) ? win_next[i] : win[i], z);
      __builtin_amdgcn_sched_barrier(0);
      own_group(2);
      if (q == 1) read_win_raw(P + kKGroups, win_next);
      __builtin_amdgcn_sched_barrier(0);
      own_group(3);
      nxt[0] = convert1(ca[0], cb[0]);
      __builtin_amdgcn_sched_barrier(0);
      oth_group(0);
      w[q][0] = load_one(P + kKGroups, q, 0);
      if constexpr (kOwn > 1) nxt[1] = convert1(ca[1], cb[1]);
      put1(buf ^ 1, 0, nxt[0]);
      __builtin_amdgcn_sched_barrier(0);
      oth_group(1);
      w[q][1] = load_one(P + kKGroups, q, 1);
      if constexpr (kOwn > 2) nxt[2] = convert1(ca[2], cb[2]);
      if constexpr (kOwn > 1) put1(buf ^ 1, 1, nxt[1]);
      if (q == 1) fix_win(win_next);
      __builtin_amdgcn_sched_barrier(0);
      oth_group(2);
      w[q][2] = load_one(P + kKGroups, q, 2);
      if constexpr (kOwn > 2) put1(buf ^ 1, 2, nxt[2]);
      __builtin_amdgcn_sched_barrier(0);
      oth_group(3);
      w[q][3] = load_one(P + kKGroups, q, 3);
      __builtin_amdgcn_sched_barrier(0);
      if (kLate && q == 0) {
        // Patch rows.  Loads return in order, and a row comes from further
        // away than the weights: its loads follow a K-step's weight loads, the
        // next weight loads come half a K-step later and are used two and a
        // half K-steps after that, and the row goes into the ring three K-steps
        // later, so that nothing waits for a row that takes less than 2 us.
        // The slot it overwrites held a row below every row that any wave
        // still reads; the barriers publish it before the step that first
        // needs it.  Block-uniform conditions.
        if (row_pending) store_row(rv, ++loaded_hi);
        row_pending = top_row(step + kAhead) > loaded_hi;
        if (row_pending) load_row(rv, loaded_hi + 1);
      }
#pragma unroll
      for (int i = 0; i < kOwn; ++i) own[i] = nxt[i];
      if (q == 2) {
#pragma unroll
        for (int i = 0; i < kOwn; ++i) win[i] = win_next[i];
        // (the slot it overwrites held a row below every row that any wave still
        // reads; first needed two steps later)
        if (!kLate && row_pending) store_row(rv, ++loaded_hi);
      }
      buf ^= 1;
      // publishes the next K-step's swap fragments (and a new row); the
      // buffer written next was last read before this barrier
      __syncthreads();
    }
  }

    // ---- fixed-order reduction over position groups, per output half:
    //      (g0 + g2) + (g1 + g3), finished by one wave per accumulator tile.
    // The four waves of an output half hold the same tiles (they share the
    // own/partner tile order); position group g finishes the g-th quarter of
    // them: with one range per block in one pass through the whole LDS, else
    // half of the quarter in each of two passes through the swap buffers and
    // the LDS behind them, so that the ring stays as it is for the next range.
    // 16 B per lane and access (conflict-free b128).
    auto tile = [&](auto qc) -> floatx4& {
      constexpr int q = decltype(qc)::value, m = q / kTiles, j = q % kTiles;
      if constexpr (j < kOwn) return acc_own[m][j];
      else return acc_oth[m][j - kOwn];
    };
    // the lane index anew: addresses derived from it stay out of the K loop's registers
    int rl = lane;
    asm volatile("" : "+v"(rl));
    float* dst = part + ((int64_t)split * n + p_base) * kFc1Out;
    // tiles o * kPer + j0 .. o * kPer + j0 + kN - 1 of every group o; the
    // src-th other group writes entry(o, j, src)
    auto reduce = [&](auto j0c, auto nc, floatx4* red) {
      constexpr int j0 = decltype(j0c)::value, kN = decltype(nc)::value;
      auto entry = [&](int o, int j, int src) {
        return (((nh * kKGroups + o) * kN + j) * (kKGroups - 1) + src) * 64 + rl;
      };
      static_for<kKGroups * kN>([&](auto ic) {
        constexpr int o = decltype(ic)::value / kN, j = decltype(ic)::value % kN;
        if (kg != o)
          red[entry(o, j, kg - (kg > o ? 1 : 0))] = tile(std::integral_constant<int, o * kPer + j0 + j>{});
      });
      __syncthreads();
      // tile q = m * kTiles + t: outputs 16(nh*kMT + m) + 4*grp + e for patch
      // 16*(block tile) + col, the block tile nh*kOwn + t (own) or
      // (1-nh)*kOwn + t - kOwn (partner's)
      static_for<kKGroups * kN>([&](auto ic) {
        constexpr int o = decltype(ic)::value / kN, j = decltype(ic)::value % kN;
        constexpr int q = o * kPer + j0 + j, m = q / kTiles, t = q % kTiles;
        if (kg == o) {
          floatx4 v[kKGroups];
#pragma unroll
          for (int g = 0; g < kKGroups; ++g)
            v[g] = (g == o) ? tile(std::integral_constant<int, q>{}) : red[entry(o, j, g - (g > o ? 1 : 0))];
          const floatx4 sum = (v[0] + v[2]) + (v[1] + v[3]);
          const int pt = ((t < kOwn) ? nh * kOwn + t : (1 - nh) * kOwn + (t - kOwn)) * 16 + (rl & 15);
          const int out = 16 * (nh * kMT + m) + 4 * (rl >> 4);
          // the partials are read once, by the tail kernel: non-temporal stores keep
          // them from evicting the FC1 weights from L2
          if (p_base + pt < n) __builtin_nontemporal_store(sum, reinterpret_cast<floatx4*>(dst + pt * kFc1Out + out));
        }
      });
    };
    if constexpr (kMulti) {
      constexpr int kPass = T::kRedTiles;
      floatx4* red = reinterpret_cast<floatx4*>(lds + T::kSwapOff);
      reduce(std::integral_constant<int, 0>{}, std::integral_constant<int, kPass>{}, red);
      __syncthreads();
      reduce(std::integral_constant<int, kPass>{}, std::integral_constant<int, kPer - kPass>{}, red);
    } else {
      reduce(std::integral_constant<int, 0>{}, std::integral_constant<int, kPer>{}, reinterpret_cast<floatx4*>(lds));
    }
    if (split + 1 < split0 + ranges) __syncthreads();
  }
}

// Blocks of a launch.  Most of a block's time outside its loop goes to its
// first patch rows, so a block takes 4 or 2 consecutive position ranges where
// whole rounds of those can be filled (us per call with one range per block and
// now: 64 requests of 235 hits 427.8 -> 420.6, 8,000 hits 226.9 -> 223.6, 16,384
// pre-cut patches 413.1 -> 401.8, 4,096 117.3 -> 115.5).  A patch's sums
// do not depend on the size of the tile it is in (every MFMA column and every
// reduction step is per patch) nor on how many ranges a block takes.  In launch
// order: big tiles with 4, 2 and 1 ranges per block, then mid tiles with 2 and 1.
struct Blocks16 {
  int64_t big4, big2, big1, mid2, mid1;      // tiles
};

template <bool kFp16, class In, bool kMulti>
__global__ __launch_bounds__(kThreads, 1) void conv_fc1_16_kernel(
    const In* __restrict__ patches, int64_t n, Blocks16 bl, const uint4* __restrict__ w1p, const uint4* __restrict__ convp,
    float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) uint32_t lds[Tile<kBigTile>::kLdsDwords];
  int64_t first = 0, t;
  int ranges = 1, split;
  bool mid;
  if constexpr (kMulti) {
    // segment of block b: 8 blocks (one per XCD) hold 1 << lr tiles, each block
    // 1 << lr ranges of one.  (In shifts, and only here: the same arithmetic with
    // 64-bit divisions cost every block about 1 us, 2,049 hits 80.4 -> 81.9 us.)
    int64_t b = blockIdx.x, tiles = bl.big4;
    int lr = 2;
    mid = false;
    auto blocks = [&] { return (tiles + (1 << lr) - 1) >> lr << 3; };
    auto next = [&](int64_t n_tiles, int l) {
      b -= blocks();
      first += tiles;
      tiles = n_tiles;
      lr = l;
    };
    if (b >= blocks()) next(bl.big2, 1);
    if (lr == 1 && b >= blocks()) next(bl.big1, 0);
    if (lr == 0 && b >= blocks()) {
      next(bl.mid2, 1);
      first = 0;
      mid = true;
      if (b >= blocks()) next(bl.mid1, 0);
    }
    // XCD x = b % 8 takes range group x % (8 / ranges): the blocks that run on
    // one XCD at a time stream the same weights through its L2
    const int x = (int)(b & 7);
    ranges = 1 << lr;
    t = (b >> 3 << lr) + (x >> (3 - lr));
    if (t >= tiles) return;
    split = (x & ((kSplits16 >> lr) - 1)) << lr;
  } else {
    split = blockIdx.x % kSplits16;
    t = blockIdx.x / kSplits16;
    mid = t >= bl.big1;
    if (mid) t -= bl.big1;
  }
  if (!mid)
    conv_fc1_block<kFp16, kBigTile, In, kMulti>(lds, split, ranges, (first + t) * kBigTile, patches, n, w1p, convp,
                                    part);
  else
    conv_fc1_block<kFp16, kMidTile, In, kMulti>(
        lds, split, ranges, (bl.big4 + bl.big2 + bl.big1) * kBigTile + (first + t) * kMidTile, patches,
        n, w1p, convp, part);
}

// The same for the hits of a batch whose tiles of 64 patches fit one round of
// the CUs: it reads the rows of the planes itself.
template <bool kFp16>
__global__ __launch_bounds__(kThreads, 1) void conv_fc1_16_hits_kernel(HitSource src, const uint4* __restrict__ w1p,
                                                                       const uint4* __restrict__ convp,
                                                                       float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) uint32_t lds[Tile<kMidTile>::kLdsDwords + kMidTile * 4];
  conv_fc1_block<kFp16, kMidTile, HitSource, false>(lds, blockIdx.x % kSplits16, 1,
                                                    (int64_t)(blockIdx.x / kSplits16) * kMidTile, &src, src.n, w1p,
                                                    convp, part);
}

// ---- Thin tiles: batches that leave most of the chip idle.  Then one block's
// K-loop is the whole call, and the barrier per K-step and the swap through
// LDS are latency, not throughput.  A thin block holds 16 or 32 patches (1 or
// 2 MFMA patch tiles) with the same 8 waves (position group x output half);
// each wave computes the conv of every tile of the block (the two output
// halves of a position group both compute it: twice the conv MFMAs, on a chip
// that is mostly idle) and feeds it to its own FC1 MFMAs, so no fragment
// crosses waves.  All input rows of the block's position range (at most 11)
// are staged in LDS once, so the loop has no barrier.  Every FC1 accumulator
// sees the same operands in the same order as in the tiles above, and the
// reduction over position groups is the same: a patch's sums are bit for bit
// those of the other tile shapes.
// With kParts = 2 or 4 the 128 FC1 outputs are shared by that many blocks
// (each wave takes 4 / kParts of the 16-output tiles): more blocks, each
// streaming a part of the position range's weights, for batches that would
// leave CUs idle; every block computes the conv.
template <bool kFp16, int kSplits, int kBt, int kParts, class Src>
__device__ __forceinline__ void thin_block(
    uint32_t* lds, int split, int opart, int64_t p_base, const Src& src,
    const uint4* __restrict__ w1p, const uint4* __restrict__ convp, float* __restrict__ part) {
  using T = Thin<kBt, kParts>;
  constexpr int kTiles = T::kTiles, kSlot = T::kSlot, kMTw = T::kMTw;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave % kKGroups;
  const int nh = wave / kKGroups;
  const int col = lane & 15;
  const int grp = lane >> 4;
  constexpr int kGroups = kPos / 2 / kKGroups;
  const int G0 = (kGroups * split) / kSplits;
  const int steps = (kGroups * (split + 1)) / kSplits - G0;
  const int P0 = kKGroups * G0;
  const int r0 = P0 / kPairsPerRow;                        // first input row of the range
  const int nrows = (P0 + kKGroups * steps - 1) / kPairsPerRow + kK - r0;
  const int64_t n = src.n;
  using Op = Op16<kFp16>;

  const __amdgpu_buffer_rsrc_t w1r = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint4*>(w1p), (short)0, (int)kWeightBytes, 0x00020000);
  const int ot0 = (opart * kNHalves + nh) * kMTw;           // the wave's first output tile
  const int voff = lane * 16 + ot0 * 1024;
  auto load_one = [&](int P, int q, int m) {
    return __builtin_bit_cast(
        uint4, __builtin_amdgcn_raw_buffer_load_b128(w1r, voff + m * 1024, (P * 3 + q) * 8 * 1024, 0));
  };
  // FC1 weights: 3 register sets, set q for K-step q of a pair, each reloaded
  // for the next pair as soon as its MFMAs have issued (three K-steps ahead:
  // with one or two patch tiles a K-step is short)
  uint4 w[3][kMTw];
  // the six conv filter fragments [shift][channel tile], kept in registers:
  // K-step q uses fragments 2q and 2q + 1
  uint4 filt[6];
  auto load_weights = [&] {
#pragma unroll
    for (int m = 0; m < kMTw; ++m) {
      w[0][m] = load_one(P0 + kg, 0, m);
      w[1][m] = load_one(P0 + kg, 1, m);
      w[2][m] = load_one(P0 + kg, 2, m);
    }
  };
  auto load_filters = [&] {
#pragma unroll
    for (int k = 0; k < 6; ++k) filt[k] = convp[k * 64 + lane];
  };
  // Loads return in order: the weights and filters first where the rows wait for
  // the hits anyway, else behind the rows
  if constexpr (std::is_same<Src, HitSource>::value) {
    load_weights();
    load_filters();
    thin_stage<kFp16, kBt, kParts>(lds, p_base, src, r0, nrows, w1p);
  } else {
    thin_stage<kFp16, kBt, kParts>(lds, p_base, src, r0, nrows, w1p);
    load_filters();
    load_weights();
  }

  int woff[4], wrow[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    int f = 8 * grp + 2 * d;
    if (f > 28) f = 28;                      // slots 30-31 are constants (set below)
    wrow[d] = f / 6 - r0;
    woff[d] = (f % 6) / 2 + col * kRP;
  }
  const bool const_slot = (grp == 3);
  auto read_win = [&](int P, uint4 (&win)[kTiles]) {
    const int y = P / kPairsPerRow;
    const int xh = P - y * kPairsPerRow;
    int base[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) base[d] = (y + wrow[d]) * kSlot + woff[d] + xh;
#pragma unroll
    for (int i = 0; i < kTiles; ++i) {
      const int o = i * 16 * kRP;
      win[i].x = lds[base[0] + o];
      win[i].y = lds[base[1] + o];
      win[i].z = lds[base[2] + o];
      win[i].w = const_slot ? Op::kOnes : lds[base[3] + o];
    }
  };
  auto convert1 = [&](const floatx4& ca, const floatx4& cb) {
    return make_uint4(relu2(Op::pack(ca[0], ca[1])), relu2(Op::pack(ca[2], ca[3])),
                      relu2(Op::pack(cb[0], cb[1])), relu2(Op::pack(cb[2], cb[3])));
  };
  floatx4 acc[kMTw][kTiles];
#pragma unroll
  for (int m = 0; m < kMTw; ++m)
#pragma unroll
    for (int i = 0; i < kTiles; ++i) acc[m][i] = (floatx4){0.f, 0.f, 0.f, 0.f};
  uint4 win[kTiles], own[kTiles];
  __syncthreads();                           // the staged rows
  const floatx4 z = {0.f, 0.f, 0.f, 0.f};
  read_win(P0 + kg, win);
#pragma unroll
  for (int i = 0; i < kTiles; ++i) own[i] = convert1(Op::mfma(filt[0], win[i], z), Op::mfma(filt[1], win[i], z));

#pragma unroll 1
  for (int step = 0; step < steps; ++step) {
    const int P = P0 + kKGroups * step + kg;
    uint4 win_next[kTiles];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int nq = (q + 1) % 3;            // the next K-step
      // FC1 of K-step q (the pair after the last one is loaded too)
#pragma unroll
      for (int m = 0; m < kMTw; ++m) {
#pragma unroll
        for (int i = 0; i < kTiles; ++i) acc[m][i] = Op::mfma(w[q][m], own[i], acc[m][i]);
        w[q][m] = load_one(P + kKGroups, q, m);
      }
      // conv of the next K-step (its window: this pair's, or the next pair's
      // after the last K-step)
      if (q == 1) read_win(P + kKGroups, win_next);
#pragma unroll
      for (int i = 0; i < kTiles; ++i) {
        const uint4& wi = (q == 2) ? win_next[i] : win[i];
        own[i] = convert1(Op::mfma(filt[2 * nq], wi, z), Op::mfma(filt[2 * nq + 1], wi, z));
      }
      if (q == 2) {
#pragma unroll
        for (int i = 0; i < kTiles; ++i) win[i] = win_next[i];
      }
    }
  }

  thin_reduce<kBt, kParts>(lds, acc, ot0, p_base, n, part + ((int64_t)split * n + p_base) * kFc1Out);
}

// Block b: split b % kSplits, then output part, then patch tile.  Src: hits, or
// pre-cut patches alone, which need no descriptors and 2.8 KB less of arguments (as
// one kernel for both, 1 patch took 18.0 us per call, now 16.5; 128 patches 21.6,
// now 20.7).
template <bool kFp16, int kSplits, int kBt, int kParts, class Src>
__global__ __launch_bounds__(kThreads, 1) void conv_fc1_16_thin_kernel(
    Src src, const uint4* __restrict__ w1p, const uint4* __restrict__ convp,
    float* __restrict__ part) {
  static_assert(thin_rows_needed(kSplits) <= kThinRows, "a position range's rows fit the stage");
  __shared__ __attribute__((aligned(16))) uint32_t lds[Thin<kBt, kParts>::kLdsDwords];
  const int split = blockIdx.x % kSplits;
  const int64_t r = blockIdx.x / kSplits;
  const int opart = (int)(r % kParts);
  const int64_t t = r / kParts;
  thin_block<kFp16, kSplits, kBt, kParts, Src>(lds, split, opart, t * kBt, src, w1p, convp, part);
}

}  // namespace

int conv_fc1_16_splits() { return kSplits16; }
int64_t conv_fc1_16_weight_bytes() { return kWeightBytes; }

// One block per CU and (tile, split), so a round of the CUs holds `per_round`
// tiles.  Whole rounds of big tiles, then the rest as rounds of mid tiles or
// of big tiles, whichever ends first by the relative round time of mid
// tiles (a 64-patch block takes about 0.72 of a 96-patch block's time: its
// weight fragments feed 4 MFMAs instead of 6).  Giving up one or two rounds
// of big tiles for rounds of mid tiles often ends sooner than a last, partly
// filled round of big tiles (B = 16,384: 4 rounds of 96 and 2 of 64 = 5.44
// against 6 rounds of 96).  (A last round of 32-patch tiles, at about 0.55 of
// a big round, never beats two rounds of mid tiles after one big round fewer;
// batches of at most one round of 32-patch tiles run thin tiles.)
void conv_fc1_16_tiles(int64_t n, int cus, int64_t* n_big, int64_t* n_mid) {
  constexpr double kRoundMid = 0.72;
  const int64_t per_round = cus >= kSplits16 ? cus / kSplits16 : 1;   // tiles per round
  const int64_t full = n / (kBigTile * per_round);
  auto rounds = [&](int64_t tiles) { return (tiles + per_round - 1) / per_round; };
  double best = 0.0;
  bool have = false;
  for (int64_t r = full; r >= 0 && r >= full - 2; --r) {
    const int64_t big = r * per_round;
    const int64_t rest = n - big * kBigTile;
    const int64_t t_mid = (rest + kMidTile - 1) / kMidTile;
    const int64_t t_big = (rest + kBigTile - 1) / kBigTile;
    auto consider = [&](double cost, int64_t b, int64_t m) {
      if (have && !(cost < best - 1e-9)) return;
      have = true;
      best = cost;
      *n_big = b;
      *n_mid = m;
    };
    consider(r + kRoundMid * (double)rounds(t_mid), big, t_mid);
    consider(r + (double)rounds(t_big), big + t_big, 0);
  }
}

// Thin tiles (16 or 32 patches) when the batch in them fills at most one
// round of the CUs: the call is then one block's K-loop long.  0: the tiles above.
int conv_fc1_16_thin_tile(int64_t n, int cus) {
  const int64_t per_round = cus >= kSplits16 ? cus / kSplits16 : 1;   // tiles per round
  if (n <= 16 * per_round) return 16;
  if (n <= 32 * per_round) return 32;
  return 0;
}

// Output parts of a 16-patch thin tile: the most (4, 2 or 1) whose blocks
// still fit one round of the CUs.  (Two blocks per CU were slower than one
// block with all the outputs: 512 patches 54.5 against 51.5 us per call,
// 1,024 in 32-patch tiles 71.6 against 60.9 us.)
int conv_fc1_16_thin_parts(int64_t n, int cus, int thin) {
  if (thin != 16) return 1;
  const int64_t blocks = (n + thin - 1) / thin * kSplits16;
  if (4 * blocks <= cus) return 4;
  return 2 * blocks <= cus ? 2 : 1;
}

// Hits the kernels read from the planes themselves: batches of thin tiles, and
// of one round of 64-patch tiles (1,025 to 2,048 patches on 256 CUs).  Such a
// call is one block long, the chip's power limit is not reached, and the
// gather's launch is what can be saved: 1,100 hits 59.7 -> 56.7 us per call, 2,048
// hits 65.7 -> 63.3.  In 96-patch tiles the row addresses leave too few
// registers: 2,600 hits 86.1 us, with the gather 82.0.
bool conv_fc1_16_direct(int64_t n, int cus) {
  if (conv_fc1_16_thin_tile(n, cus)) return true;
  int64_t n_big = 0, n_mid = 0;
  conv_fc1_16_tiles(n, cus, &n_big, &n_mid);
  return n_big == 0 && n_mid * kSplits16 <= cus;
}

template <bool kFp16>
hipError_t launch_typed(const RowInput& in, int64_t n, const uint4* w1p, const uint4* convp,
                        float* part, int cus, hipStream_t stream) {
  const int thin = conv_fc1_16_thin_tile(n, cus);
  if (thin) {
    const int parts = conv_fc1_16_thin_parts(n, cus, thin);
    const dim3 grid((unsigned)((n + thin - 1) / thin * kSplits16 * parts));
    auto run = [&](const auto& src) {
      using Src = std::decay_t<decltype(src)>;
      auto go = [&](auto kernel) {
        return launch_kernel(kernel, grid, dim3(kThreads), 0, stream, src, w1p, convp, part);
      };
      if (thin == 32) return go(conv_fc1_16_thin_kernel<kFp16, kSplits16, 32, 1, Src>);
      if (parts == 4) return go(conv_fc1_16_thin_kernel<kFp16, kSplits16, 16, 4, Src>);
      return parts == 2 ? go(conv_fc1_16_thin_kernel<kFp16, kSplits16, 16, 2, Src>)
                        : go(conv_fc1_16_thin_kernel<kFp16, kSplits16, 16, 1, Src>);
    };
    return in.patches ? run(PatchSource{in.patches, n}) : run(hit_source(in, n));
  }
  int64_t n_big = 0, n_mid = 0;
  conv_fc1_16_tiles(n, cus, &n_big, &n_mid);
  if (!in.patches && !in.patches16)
    return launch_kernel(conv_fc1_16_hits_kernel<kFp16>, dim3((unsigned)(n_mid * kSplits16)), dim3(kThreads), 0, stream,
                         hit_source(in, n), w1p, convp, part);
  // blocks of several ranges for the whole rounds of tiles there are
  const int64_t round = cus >= kSplits16 ? cus / kSplits16 : 1;
  Blocks16 bl = {};
  bl.big4 = n_big / (4 * round) * (4 * round);
  bl.big2 = (n_big - bl.big4) / (2 * round) * (2 * round);
  bl.big1 = n_big - bl.big4 - bl.big2;
  bl.mid2 = n_mid / (2 * round) * (2 * round);
  if (n_mid - bl.mid2 > round) bl.mid2 = n_mid;
  bl.mid1 = n_mid - bl.mid2;
  const int64_t blocks = bl.big4 * 2 + bl.big2 * 4 + bl.big1 * 8 + (bl.mid2 + 1) / 2 * 8 + bl.mid1 * 8;
  auto go = [&](auto kernel, auto* patches) {
    return launch_kernel(kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream, patches, n, bl, w1p,
                         convp, part);
  };
  const bool multi = bl.big4 + bl.big2 + bl.mid2 > 0;
  if (in.patches)
    return multi ? go(conv_fc1_16_kernel<kFp16, float, true>, in.patches)
                 : go(conv_fc1_16_kernel<kFp16, float, false>, in.patches);
  return multi ? go(conv_fc1_16_kernel<kFp16, uint16_t, true>, in.patches16)
               : go(conv_fc1_16_kernel<kFp16, uint16_t, false>, in.patches16);
}

hipError_t launch_conv_fc1_16(bool fp16, const RowInput& in, int64_t n, const uint4* w1p,
                              const uint4* convp, float* part, int cus, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  return fp16 ? launch_typed<true>(in, n, w1p, convp, part, cus, stream)
              : launch_typed<false>(in, n, w1p, convp, part, cus, stream);
}

}  // namespace pointid
