// The parts that the thin tiles of the 16-bit and the 8-bit fused conv/FC1
// kernels share: blocks of 16 or 32 patches for batches that leave most of the
// chip idle (see conv_fc1_16.hip), their patch rows and their reduction.
#pragma once

#include "internal.h"
#include "op16.h"
#include "rows.h"

namespace pointid {
namespace {

constexpr int kKGroups = 4;                   // position groups (interleaved pairs)
constexpr int kNHalves = 2;                   // output halves
constexpr int kWaves = kKGroups * kNHalves;   // 8
constexpr int kThreads = kWaves * 64;         // 512
constexpr int kMT = 8 / kNHalves;             // 16-output tiles per wave
constexpr int kPairsPerRow = kFm / 2;         // 22
constexpr int kRP = 26;                       // LDS row pitch, dwords (24 used)

constexpr int kThinRows = 11;                 // input rows of one position range, at most
template <int kBt, int kParts>
struct Thin {
  static constexpr int kTiles = kBt / 16;
  static constexpr int kMTw = kMT / kParts;                // 16-output tiles per wave
  static constexpr int kSlot = kBt * kRP;                  // dwords per staged row
  // the reduction: per output half, 3 tiles from the other groups per accumulator tile
  static constexpr int kRed = kNHalves * kMTw * kTiles * (kKGroups - 1) * 4 * 64;
  // one row slot more than a range needs: the loop reads the window of the
  // pair after its last one (the result is never used), which may lie one row lower
  static constexpr int kRowsDw = (kThinRows + 1) * kSlot;
  static constexpr int kDescOff = kRowsDw;                 // the block's row descriptors
  static constexpr int kMain = kDescOff + kBt * 4;
  static constexpr int kLdsDwords = kMain > kRed ? kMain : kRed;
  static constexpr int kRowAll = kBt * kRowChunks;         // 4-pixel chunks per staged row
  static constexpr int kPer = (kThinRows * kRowAll + kThreads - 1) / kThreads;
  static_assert(kTiles >= 1 && kTiles <= 2, "1 or 2 patch tiles");
  static_assert(kParts == 1 || kParts == 2 || kParts == 4, "whole, half or quarter of the outputs");
};

// input rows a position range spans, at most, over the ranges of `splits`
constexpr int thin_rows_needed(int splits) {
  int most = 0;
  for (int s = 0; s < splits; ++s) {
    const int g0 = (kPos / 2 / kKGroups) * s / splits;
    const int g1 = (kPos / 2 / kKGroups) * (s + 1) / splits;
    const int rows = (kKGroups * g1 - 1) / kPairsPerRow + kK - (kKGroups * g0) / kPairsPerRow;
    most = rows > most ? rows : most;
  }
  return most;
}

// Every input row of a position range (rows r0 .. r0 + nrows - 1 of the block's
// patches), rounded to 16 bits, into LDS, all loads in flight together.  `safe`:
// any 16 readable bytes.
template <bool kFp16, int kBt, int kParts>
__device__ __forceinline__ void thin_stage(uint32_t* lds, int64_t p_base, const HitSource& src, int r0, int nrows,
                                           const void* safe) {
  using T = Thin<kBt, kParts>;
  using Op = Op16<kFp16>;
  constexpr int kSlot = T::kSlot;
  const int tid = threadIdx.x;
  uint4* desc = reinterpret_cast<uint4*>(lds + T::kDescOff);
  if (tid < kBt) desc[tid] = src.get(p_base + tid);
  __syncthreads();
  const int total = nrows * T::kRowAll;
  rowx4 v[T::kPer];
  uint32_t kinds = 0;                      // 2 bits per chunk
  static_assert(2 * T::kPer <= 32, "kinds");
#pragma unroll
  for (int k = 0; k < T::kPer; ++k) {
    const int c = tid + k * kThreads;
    if (c < total) {
      const int j = c / T::kRowAll, cc = c - j * T::kRowAll;
      uint32_t kind;
      v[k] = row_chunk_load(desc_from_lds(desc + cc / kRowChunks), r0 + j,
                            cc - (cc / kRowChunks) * kRowChunks, safe, &kind);
      kinds |= kind << 2 * k;
    }
  }
#pragma unroll
  for (int k = 0; k < T::kPer; ++k) {
    const int c = tid + k * kThreads;
    if (c < total) {
      const int j = c / T::kRowAll, cc = c - j * T::kRowAll;
      const int p = cc / kRowChunks, h = cc - (cc / kRowChunks) * kRowChunks;
      const rowx4 x = row_chunk_finish(desc + p, r0 + j, h, v[k], (kinds >> 2 * k) & 3);
      *reinterpret_cast<uint2*>(lds + j * kSlot + p * kRP + h * 2) =
          make_uint2(Op::pack(x[0], x[1]), Op::pack(x[2], x[3]));
    }
  }
}

// The same for pre-cut patches: no descriptors, no barrier behind them, 8 pixels a
// thread and turn (patches past the batch: its last one, never stored).  `safe`
// is not needed.
template <bool kFp16, int kBt, int kParts>
__device__ __forceinline__ void thin_stage(uint32_t* lds, int64_t p_base, const PatchSource& src, int r0, int nrows,
                                           const void*) {
  using Op = Op16<kFp16>;
  constexpr int kChunks = kPatch / 8, kRow = kBt * kChunks, kPer = (kThinRows * kRow + kThreads - 1) / kThreads;
  const int tid = threadIdx.x, total = nrows * kRow;
  rowx4 v[kPer][2];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int c = tid + k * kThreads;
    if (c < total) {
      const int j = c / kRow, cc = c - j * kRow, p = cc / kChunks, h = cc - p * kChunks;
      const int64_t at = p_base + p < src.n ? p_base + p : src.n - 1;
      const rowx4* from = reinterpret_cast<const rowx4*>(src.patches + at * kPatchPix + (r0 + j) * kPatch + 8 * h);
      v[k][0] = __builtin_nontemporal_load(from);
      v[k][1] = __builtin_nontemporal_load(from + 1);
    }
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int c = tid + k * kThreads;
    if (c < total) {
      const int j = c / kRow, cc = c - j * kRow, p = cc / kChunks, h = cc - p * kChunks;
      uint32_t* d = lds + j * Thin<kBt, kParts>::kSlot + p * kRP + h * 4;
#pragma unroll
      for (int i = 0; i < 2; ++i)
        *reinterpret_cast<uint2*>(d + 2 * i) =
            make_uint2(Op::pack(v[k][i][0], v[k][i][1]), Op::pack(v[k][i][2], v[k][i][3]));
    }
  }
}

// The fixed-order reduction (g0 + g2) + (g1 + g3) over the position groups of a
// thin block, and its store to part[.][p_base ..] (`dst`: the block's first
// patch): each position group finishes a quarter of its output half's tiles
// (with 2 tiles per half groups 0 and 2 finish one each, with 1 group 0
// finishes it).  ot0: the wave's first output tile; n - p_base patches exist.
template <int kBt, int kParts>
__device__ __forceinline__ void thin_reduce(uint32_t* lds, floatx4 (&acc)[Thin<kBt, kParts>::kMTw][Thin<kBt, kParts>::kTiles],
                                            int ot0, int64_t p_base, int64_t n, float* __restrict__ dst) {
  using T = Thin<kBt, kParts>;
  constexpr int kTiles = T::kTiles, kMTw = T::kMTw;
  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wave % kKGroups, nh = wave / kKGroups;
  __syncthreads();                           // every wave is done with the rows
  constexpr int kSlots = kMTw * kTiles;
  static_assert(kSlots % kKGroups == 0 || kKGroups % kSlots == 0, "tiles spread evenly");
  // the position group that finishes slot q
  constexpr auto owner = [](int q) {
    return kSlots >= kKGroups ? q / (kSlots / kKGroups) : q * (kKGroups / kSlots);
  };
  floatx4* red = reinterpret_cast<floatx4*>(lds);
  auto entry = [&](int q, int src) { return ((nh * kSlots + q) * (kKGroups - 1) + src) * 64 + lane; };
  auto tile = [&](auto qc) -> floatx4& {
    constexpr int q = decltype(qc)::value;
    return acc[q / kTiles][q % kTiles];
  };
  static_for<kSlots>([&](auto qc) {
    constexpr int o = owner(decltype(qc)::value);
    if (kg != o) red[entry(decltype(qc)::value, kg - (kg > o ? 1 : 0))] = tile(qc);
  });
  __syncthreads();

  static_for<kSlots>([&](auto qc) {
    constexpr int q = decltype(qc)::value, o = owner(q), m = q / kTiles, i = q % kTiles;
    if (kg == o) {
      floatx4 v[kKGroups];
#pragma unroll
      for (int g = 0; g < kKGroups; ++g)
        v[g] = (g == o) ? tile(qc) : red[entry(q, g - (g > o ? 1 : 0))];
      const floatx4 sum = (v[0] + v[2]) + (v[1] + v[3]);
      const int64_t po = (int64_t)i * 16 + col;
      const int out = 16 * (ot0 + m) + 4 * grp;
      if (p_base + po < n)
        __builtin_nontemporal_store(sum, reinterpret_cast<floatx4*>(dst + po * kFc1Out + out));
    }
  });
}

}  // namespace
}  // namespace pointid
