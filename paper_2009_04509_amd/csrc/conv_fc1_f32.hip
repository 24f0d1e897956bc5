// Fused conv 5x5 (1->48) + ReLU + FC1 (92928->128) in fp32 on the fp32 MFMA
// (v_mfma_f32_16x16x4_f32), paper §2.2: the fp32 path.  The conv maps exist
// only in registers and LDS, and the patch rows are read from the plane images
// or the pre-cut patches themselves (rows.h): no patch is written and read back.
//
// Arithmetic.  Map positions go in pairs (x, x+1), x even, in 8 contiguous
// ranges (split-K) of 4 interleaved position groups (group g takes the pairs
// 4k + g of a range).  The 5x6 window of a pair (30 pixels), a constant 1.0 for
// the bias and a zero fill the K = 32 conv operand, taken as 8 MFMAs of K = 4
// (slot f = 4i + g for MFMA i and lane group g).  Its 6 conv tiles (2 shifts x
// 3 channel tiles of 16) are the pair's 6 K-steps.  Per K-step q (shift s,
// channel tile t) and 16-patch tile:
//   conv:  C[ch][patch] = sum_f Kc[ch][f] * Win[f][patch] (8 MFMAs); lane
//          (col, g) ends with channels 16t + 4g + e, e = 0..3, of patch col;
//   FC1:   chunk e uses that value as B operand K-slot g, so K-slot g of chunk
//          e is FC1 input (y*44 + x + s)*48 + 16t + 4g + e; the weights are
//          packed in that order, one 1 KiB fragment per (pair, K-step, 16 outputs).
// A patch's sums are one chain of MFMAs per range and group, added as
// (g0 + g2) + (g1 + g3): they do not depend on the shape of the block.
//
// Work split.  8 waves share a position group, one per 16 outputs: the wave
// holds one accumulator tile per patch tile and streams the FC1 weights of its
// outputs.  The conv tiles of a pair are shared out over the 8 waves (so that
// every SIMD computes as many), which read each other's through LDS: the conv
// is computed once per block and there is one barrier per pair.  The input rows
// of the range (at most 11) are staged in LDS at the start.  A block takes
//   2 patch tiles (32 patches) and all 4 groups, two at a time by two sets of
//     8 waves (16 waves, 4 per SIMD; 139 KB of LDS), in whole rounds;
//   1 patch tile and all 4 groups, for a last round that is at most half full;
//   1 patch tile and one group (8 waves, two such blocks fit a CU), for batches
//     that would leave CUs idle otherwise: the groups' sums go to the tail.
// Bound by the fp32 MFMA: 240 MFMAs per pair and patch tile against 48 weight
// loads, 48 fragment reads and 48 window reads.
#include "internal.h"
#include "rows.h"

namespace pointid {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kGroups = 4;                    // position groups
constexpr int kSplits = 8;                    // position ranges
constexpr int kMTiles = kFc1Out / 16;         // 16-output tiles: the waves of a group
constexpr int kSet = kMTiles * 64;            // threads of a group
constexpr int kRP = 52;                       // LDS row pitch (dwords; 48 used)
constexpr int kPairsPerRow = kFm / 2;         // 22
constexpr int kPairs = kPos / 2;              // 968
constexpr int kQ = 6;                         // K-steps per pair (2 shifts x 3 channel tiles)
constexpr int kRows = 11;                     // input rows of one range, at most
static_assert(kPairs % kGroups == 0, "whole steps");

// first step (kGroups pairs) of range s, of 242 in all
__host__ __device__ constexpr int range_begin(int s) { return kPairs / kGroups * s / kSplits; }
constexpr int rows_needed() {
  int most = 0;
  for (int s = 0; s < kSplits; ++s) {
    const int p0 = kGroups * range_begin(s), p1 = kGroups * range_begin(s + 1) - 1;
    const int rows = p1 / kPairsPerRow + kK - p0 / kPairsPerRow;
    most = rows > most ? rows : most;
  }
  return most;
}
static_assert(rows_needed() <= kRows, "a range's rows fit the stage");

// LDS of a block (dwords): rows | conv tiles [2 buffers][sets][6][patch tiles]
// [64 lanes] x 4 | row descriptors.
template <int kTiles, int kSets>
struct Block {
  static constexpr int kBt = 16 * kTiles;
  static constexpr int kThreads = kSet * kSets;
  static constexpr int kSlot = kBt * kRP;                  // dwords per staged row
  static constexpr int kMapOff = kRows * kSlot;
  static constexpr int kMapBuf = kQ * kTiles * 256;        // one set's buffer
  static constexpr int kDescOff = kMapOff + 2 * kSets * kMapBuf;
  static constexpr int kLds = kDescOff + kBt * 4;
  static constexpr int kRowAll = kBt * kRowChunks;         // chunks per staged row
  static constexpr int kPer = (kRows * kRowAll + kThreads - 1) / kThreads;
  static_assert(kLds * 4 <= 160 * 1024 && 2 * kPer <= 32 && kBt <= kThreads, "block");
};

__device__ __forceinline__ floatx4 mfma4(float a, float b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// One block: patches p_base .. p_base + 16 kTiles - 1 (those past the batch
// hold zeros and are not stored), range `split`; kSets sets of 8 waves take
// the groups set + g0, set + g0 + 2, ... (kSeq of them) one after the other.
// `out` points at the sums of the block's first patch.
template <int kTiles, int kSets, int kSeq>
__device__ __forceinline__ void conv_fc1_f32_block(float* lds, int split, int g0, int64_t p_base,
                                                   const HitSource& src,
                                                   const float* __restrict__ conv_w,
                                                   const float* __restrict__ conv_b,
                                                   const float* __restrict__ w1f,
                                                   float* __restrict__ out) {
  using B = Block<kTiles, kSets>;
  constexpr int kSlot = B::kSlot;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int set = wave / kMTiles, m = wave % kMTiles;
  const int col = lane & 15, grp = lane >> 4;
  const int P0 = kGroups * range_begin(split);
  const int steps = range_begin(split + 1) - range_begin(split);
  const int r0 = P0 / kPairsPerRow;                        // first input row of the range
  const int nrows = (P0 + kGroups * steps - 1) / kPairsPerRow + kK - r0;
  const int total = kSeq * steps;
  // pair i of this wave's sequence
  auto pair = [&](int i) {
    const int ph = kSeq > 1 && i >= steps ? 1 : 0;
    return P0 + kGroups * (i - ph * steps) + g0 + set + 2 * ph;
  };

  // FC1 weights of this wave's outputs: one fragment per pair and K-step,
  // reloaded for the next pair as soon as its MFMAs have issued (reads past the
  // end return 0)
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(w1f), (short)0, (int)(sizeof(float) * kFc1Out * kFc1In), 0x00020000);
  auto load_w = [&](int P, int q) {
    return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                                           wr, lane * 16, ((P * kQ + q) * kMTiles + m) * 1024, 0));
  };
  floatx4 w[kQ];
#pragma unroll
  for (int q = 0; q < kQ; ++q) w[q] = load_w(pair(0), q);

  // The conv tiles (jobs) this wave computes of a pair, job = K-step * kTiles +
  // patch tile.  2 patch tiles: job m always, and of jobs 8-11 one in every
  // other pair (waves 0-3 and 4-7 in turn); 1 patch tile: waves 0-5 and 7-2 in
  // turn.  Waves w and w + 4 share a SIMD: each SIMD computes as many.
  auto job_of = [&](int odd, int k) {        // k-th job of an even / odd pair, or -1
    if (kTiles == 2) {
      if (k == 0) return m;
      return (m < 4) == (odd == 0) ? 8 + m % 4 : -1;
    }
    if (k == 1) return -1;
    return odd == 0 ? (m < kQ ? m : -1) : (m >= kMTiles - kQ ? kMTiles - 1 - m : -1);
  };
  // Their filters, lane (channel 16t + col, K-slot group grp), MFMA i.  Two
  // sets: 2 patch tiles, the first and the second job; 1, even and odd pairs.
  float filt[2][8];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int job = kTiles == 2 ? (k == 0 ? m : 8 + m % 4) : job_of(k, 0);
    const int q = job < 0 ? 0 : job / kTiles, s = q / 3, ch = 16 * (q % 3) + col;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int f = 4 * i + grp, u = f / 6, c = f - 6 * (f / 6) - s;
      float v = 0.f;
      if (f < 30 && c >= 0 && c < kK) v = conv_w[ch * kK * kK + u * kK + c];
      if (f == 30) v = conv_b[ch];
      filt[k][i] = v;
    }
  }

  // ---- every input row of the range, all loads in flight together
  {
    uint4* desc = reinterpret_cast<uint4*>(lds + B::kDescOff);
    if (tid < B::kBt) desc[tid] = src.get(p_base + tid);
    __syncthreads();
    const int chunks = nrows * B::kRowAll;
    rowx4 v[B::kPer];
    uint32_t kinds = 0;                      // 2 bits per chunk
#pragma unroll
    for (int k = 0; k < B::kPer; ++k) {
      const int c = tid + k * B::kThreads;
      if (c < chunks) {
        const int j = c / B::kRowAll, cc = c - j * B::kRowAll;
        uint32_t kind;
        v[k] = row_chunk_load(desc_from_lds(desc + cc / kRowChunks), r0 + j,
                              cc - (cc / kRowChunks) * kRowChunks, w1f, &kind);
        kinds |= kind << 2 * k;
      }
    }
#pragma unroll
    for (int k = 0; k < B::kPer; ++k) {
      const int c = tid + k * B::kThreads;
      if (c < chunks) {
        const int j = c / B::kRowAll, cc = c - j * B::kRowAll;
        const int p = cc / kRowChunks, h = cc - (cc / kRowChunks) * kRowChunks;
        const rowx4 x = row_chunk_finish(desc + p, r0 + j, h, v[k], (kinds >> 2 * k) & 3);
        *reinterpret_cast<rowx4*>(lds + j * kSlot + p * kRP + 4 * h) = x;
      }
    }
  }
  __syncthreads();

  // this lane's window pixels: slot f = 4i + grp of patch col
  int woff[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    int f = 4 * i + grp;
    if (f > 29) f = 29;                      // slots 30-31 are constants (set below)
    woff[i] = f / 6 * kSlot + f % 6 + col * kRP;
  }
  auto read_win = [&](int P, int tile, float (&win)[8]) {
    const int y = P / kPairsPerRow;
    const int base = (y - r0) * kSlot + 2 * (P - y * kPairsPerRow) + tile * 16 * kRP;
#pragma unroll
    for (int i = 0; i < 8; ++i) win[i] = lds[base + woff[i]];
    if (grp >= 2) win[7] = grp == 2 ? 1.f : 0.f;
  };
  auto conv = [&](const float (&fr)[8], const float (&win)[8]) {
    floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) c = mfma4(fr[i], win[i], c);
    return (floatx4){fmaxf(c[0], 0.f), fmaxf(c[1], 0.f), fmaxf(c[2], 0.f), fmaxf(c[3], 0.f)};
  };
  floatx4* maps = reinterpret_cast<floatx4*>(lds + B::kMapOff) + set * 2 * (B::kMapBuf / 4) + lane;
  auto map_at = [&](int buf, int job) { return maps + (buf * kQ * kTiles + job) * 64; };

  // the jobs of the first pair
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int job = job_of(0, k);
    if (job >= 0) {
      float win[8];
      read_win(pair(0), job % kTiles, win);
      *map_at(0, job) = conv(filt[kTiles == 2 ? k : 0], win);
    }
  }
  __syncthreads();

  floatx4 acc[kTiles], sum[kTiles];
#pragma unroll
  for (int j = 0; j < kTiles; ++j) acc[j] = sum[j] = (floatx4){0.f, 0.f, 0.f, 0.f};

  // One pair: its FC1, and the jobs of the next pair (`odd`: the next pair's
  // parity) into the other buffer.
  auto step = [&](int i, auto oddc) {
    constexpr int odd = decltype(oddc)::value;
    const int Pn = pair(i + 1);
    const int job0 = job_of(odd, 0), job1 = job_of(odd, 1);
    const bool more = i + 1 < total;
    const bool do0 = more && job0 >= 0, do1 = more && job1 >= 0;   // wave-uniform
    floatx4 b[kTiles][kQ];
    auto get = [&](int q) {
#pragma unroll
      for (int j = 0; j < kTiles; ++j) b[j][q] = *map_at(odd ^ 1, q * kTiles + j);
    };
    auto fc1 = [&](int q) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < kTiles; ++j) acc[j] = mfma4(w[q][e], b[j][q][e], acc[j]);
      w[q] = load_w(Pn, q);
    };
    float win[8];
    get(0);
    get(1);
    if (do0) read_win(Pn, job0 % kTiles, win);
    fc1(0);
    get(2);
    get(3);
    if (do0) *map_at(odd, job0) = conv(filt[kTiles == 2 ? 0 : odd], win);
    fc1(1);
    if (kTiles == 2 && do1) read_win(Pn, job1 % kTiles, win);
    fc1(2);
    get(4);
    get(5);
    if (kTiles == 2 && do1) *map_at(odd, job1) = conv(filt[1], win);
    fc1(3);
    fc1(4);
    fc1(5);
    __syncthreads();
  };
  // the second group of a set starts with fresh accumulators
  auto next_group = [&](int i) {
    if (kSeq > 1 && i == steps) {
#pragma unroll
      for (int j = 0; j < kTiles; ++j) {
        sum[j] = acc[j];
        acc[j] = (floatx4){0.f, 0.f, 0.f, 0.f};
      }
    }
  };
  int i = 0;
#pragma unroll 1
  for (; i + 1 < total; i += 2) {
    next_group(i);
    step(i, std::integral_constant<int, 1>{});
    next_group(i + 1);
    step(i + 1, std::integral_constant<int, 0>{});
  }
  if (i < total) {
    next_group(i);
    step(i, std::integral_constant<int, 1>{});
  }

  // ---- fixed-order sum of the groups: (g0 + g2) + (g1 + g3)
#pragma unroll
  for (int j = 0; j < kTiles; ++j) acc[j] = kSeq > 1 ? sum[j] + acc[j] : acc[j];
  if constexpr (kSets > 1) {
    floatx4* red = reinterpret_cast<floatx4*>(lds);        // the rows are dead
    if (set == 1)
#pragma unroll
      for (int j = 0; j < kTiles; ++j) red[(m * kTiles + j) * 64 + lane] = acc[j];
    __syncthreads();
    if (set == 1) return;
#pragma unroll
    for (int j = 0; j < kTiles; ++j) acc[j] = acc[j] + red[(m * kTiles + j) * 64 + lane];
  }
  // outputs 16m + 4 grp + e of patch 16 j + col
#pragma unroll
  for (int j = 0; j < kTiles; ++j) {
    const int p = 16 * j + col;
    if (p_base + p < src.n)
      __builtin_nontemporal_store(acc[j], reinterpret_cast<floatx4*>(out + p * kFc1Out + 16 * m + 4 * grp));
  }
}

// Tiles t < n_big hold 32 patches, the ones after them 16; block b takes range
// b % 8 (one per XCD, whose L2 the blocks that run on it share for the weights).
__global__ __launch_bounds__(2 * kSet, 1) void conv_fc1_f32_kernel(
    HitSource src, int64_t n_big, const float* __restrict__ conv_w, const float* __restrict__ conv_b,
    const float* __restrict__ w1f, float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) float lds[Block<2, 2>::kLds];
  const int split = blockIdx.x % kSplits;
  const int64_t t = blockIdx.x / kSplits;
  const int64_t p = t < n_big ? t * 32 : n_big * 32 + (t - n_big) * 16;
  float* out = part + ((int64_t)split * src.n + p) * kFc1Out;
  if (t < n_big)
    conv_fc1_f32_block<2, 2, 2>(lds, split, 0, p, src, conv_w, conv_b, w1f, out);
  else
    conv_fc1_f32_block<1, 2, 2>(lds, split, 0, p, src, conv_w, conv_b, w1f, out);
}

// Small batches: a block per 16 patches, range and group; the sums of range s
// and group g go to part[4 s + g].
__global__ __launch_bounds__(kSet, 2) void conv_fc1_f32_small_kernel(
    HitSource src, const float* __restrict__ conv_w, const float* __restrict__ conv_b,
    const float* __restrict__ w1f, float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) float lds[Block<1, 1>::kLds];
  const int split = blockIdx.x % kSplits, g = blockIdx.x / kSplits % kGroups;
  const int64_t p = (int64_t)(blockIdx.x / (kSplits * kGroups)) * 16;
  conv_fc1_f32_block<1, 1, 1>(lds, split, g, p, src, conv_w, conv_b, w1f,
                              part + ((int64_t)(split * kGroups + g) * src.n + p) * kFc1Out);
}

// FC1 weights in the order the kernel reads them, once at create: one thread
// per (pair, K-step, 16 outputs, lane (output i, K-slot group g)).
__global__ __launch_bounds__(256) void pack_fc1_f32_kernel(const float* __restrict__ w1,
                                                           floatx4* __restrict__ out) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)kPairs * kQ * kMTiles * 64) return;
  const int lane = (int)(idx & 63), m = (int)(idx >> 6) % kMTiles;
  const int64_t pq = idx >> 9;
  const int q = (int)(pq % kQ);
  const int64_t k = (2 * (pq / kQ) + q / 3) * kCh + 16 * (q % 3) + 4 * (lane >> 4);
  const int o = 16 * m + (lane & 15);
  out[idx] = (floatx4){w1[k * kFc1Out + o], w1[(k + 1) * kFc1Out + o], w1[(k + 2) * kFc1Out + o],
                       w1[(k + 3) * kFc1Out + o]};
}

}  // namespace

// Position groups whose sums a launch over n patches leaves to the tail: 4 for
// small batches, 1 else.  In units of one group of one 16-patch tile on a CU,
// the small kernel takes a unit per block, the others 4 (16 patches) and 8
// (32 patches) per round of the CUs, one block each.
int conv_fc1_f32_groups(int64_t n, int cus) {
  const int64_t tiles = (n + 15) / 16;
  if (tiles > 64) return 1;
  auto rounds = [&](int64_t blocks) { return (blocks + cus - 1) / cus; };
  const int64_t small = rounds(tiles * kSplits * kGroups);
  const int64_t one = 4 * rounds(tiles * kSplits), two = 8 * rounds((tiles + 1) / 2 * kSplits);
  return small < (one < two ? one : two) ? kGroups : 1;
}
int conv_fc1_f32_splits() { return kSplits; }

// Tiles of 32 patches fill whole rounds of the CUs (one block per CU); the
// rest is cut into tiles of 16 when those fit in one round.
void conv_fc1_f32_tiles(int64_t n, int cus, int64_t* n_big, int64_t* n_small) {
  const int64_t per_round = cus >= kSplits ? cus / kSplits : 1;     // tiles per round
  int64_t big = n / (32 * per_round) * per_round;
  const int64_t rest = n - big * 32;
  int64_t small = (rest + 15) / 16;
  if (small > per_round) {
    big += (rest + 31) / 32;
    small = 0;
  }
  *n_big = big;
  *n_small = small;
}

hipError_t launch_pack_fc1_f32(const float* w1, float* w1f, hipStream_t stream) {
  const int64_t threads = (int64_t)kPairs * kQ * kMTiles * 64;
  static_assert(kPairs * kQ * kMTiles * 64 * 4 == kFc1In * kFc1Out, "every weight once");
  return launch_kernel(pack_fc1_f32_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, stream,
                       w1, reinterpret_cast<floatx4*>(w1f));
}

hipError_t launch_conv_fc1_f32(const RowInput& in, int64_t n, const float* conv_w, const float* conv_b,
                               const float* w1f, float* part, int cus, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const HitSource src = hit_source(in, n);
  if (conv_fc1_f32_groups(n, cus) > 1)
    return launch_kernel(conv_fc1_f32_small_kernel, dim3((unsigned)((n + 15) / 16 * kSplits * kGroups)),
                         dim3(kSet), 0, stream, src, conv_w, conv_b, w1f, part);
  int64_t n_big = 0, n_small = 0;
  conv_fc1_f32_tiles(n, cus, &n_big, &n_small);
  return launch_kernel(conv_fc1_f32_kernel, dim3((unsigned)((n_big + n_small) * kSplits)), dim3(2 * kSet), 0,
                       stream, src, n_big, conv_w, conv_b, w1f, part);
}

}  // namespace pointid
