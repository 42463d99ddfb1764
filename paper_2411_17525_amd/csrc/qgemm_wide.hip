// Lookup-table GEMM for HIGGS layers at prompt-sized batches (more than 64
// rows; fewer for small groups, use_qgemm_wide) on the matrix cores: the product of qgemm.hip,
//   y[b][o] = sum_i scale[o][i] * sum_j < G[code(o,i,j)], x_rot[b, ig+jp : ig+(j+1)p] >,
// in blocks of 128 or 256 rows x 64 or 128 batch columns instead of one launch
// per 64 columns. Measured on MI355X against the 64-column launches (rotated
// fp32 input): 28672 x 4096 at 2048 rows 939 -> 504 us (0.95 PFLOP/s; a plain
// fp16 product of that size in torch: 427 us), 4096 x 14336 with 10-bit codes
// at 512 rows 215 -> 110 us, 11003 x 5120 at 300 rows 150 -> 98 us.
//   * xprep_wide_kernel converts (and rotates) the activations once, to fp16
//     with one power of two per (batch row, scale group), in the layout the
//     product stages: per 256-row chunk, per 64 weights of K, one 128-byte
//     row per batch row whose 16-byte pieces are permuted by the row's low
//     bits, so that a stage goes to LDS as it lies in memory and is read back
//     as matrix operands without bank conflicts.
//   * qgemm_wide_kernel: 4 waves (one per SIMD, 512 registers), each owning 64
//     rows x 128 columns of the block, or 8 (two per SIMD) with 64 x 64 each.
//     Activation stages of 64 weights go straight from memory to LDS (no
//     registers), three buffers deep; codes are read in the operand layout two
//     stages at a time and turned into fp16 operands through the replicated
//     LDS table as in qgemm.hip.
// Scale groups: a group's sums start at zero and are added, times scale and
// activation exponent, to fp32 totals at its end, as in qgemm.hip (one
// rounding). Sums and totals of 64 x 128 take half of one wave's registers, so
// that two such waves per SIMD have no room for the totals. One running sum
// per wave, rescaled by the ratio of the scales at each group's end, let 8 of
// them work a 256 x 256 block and was 7% faster at 2048 rows (470 us), but its
// sums had about three times the rounding error.

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.h"
#include "qgemm_common.h"
#include "wave_fwht.h"

namespace higgs {
namespace {

constexpr int kChunk = 256;  // batch rows per chunk of the fp16 activations
constexpr int kBufs = 3;     // activation stages in LDS

typedef __attribute__((address_space(3))) void lds_void;
// (left to itself the compiler calls the product's larger pieces as functions
// and keeps the sums in memory)
#define HIGGS_INLINE __attribute__((always_inline))

// ---------------------------------------------------------------------------
// Activations -> fp16 and one power of two per (batch row, group).
// ---------------------------------------------------------------------------
// 16-byte piece c (8 weights) of batch row r, stage s of a chunk of R rows:
// byte ((s R + r) 8 + (c ^ (r & 7))) 16 of the chunk.
__device__ inline int64_t xw_index(int64_t batch, int64_t in, int64_t row, int64_t k) {
  const int64_t chunk = row / kChunk, r = row - chunk * kChunk;
  const int64_t rows = batch - chunk * kChunk < kChunk ? batch - chunk * kChunk : kChunk;
  return chunk * kChunk * in + (((k >> 6) * rows + r) * 8 + (((k >> 3) & 7) ^ (r & 7))) * 8 +
         (k & 7);
}

// The power of two that a group's fp16 values are in units of, as in qgemm.hip:
// the group's largest magnitude m lies in [2^14, 2^15), so that fp16 keeps all
// its bits down to 2^-28 of it.
__device__ inline int group_exponent(float m) {
  const int e = m > 0.f ? ilogbf(m) - 14 : 0;
  return e < -126 ? -126 : (e > 127 ? 127 : e);
}

// One wave per group of g = 64 E elements, W waves per block. Bound by the
// latency of one load, rotation and store per wave and by the signs that each
// block makes (two 64-bit products per sign), so 16 waves share them and a
// wave's first load is under way meanwhile: 2048 x 4096 bf16 into two layers'
// copies 27.6 -> 22.3 us against blocks of four waves that load afterwards
// (38 us with four waves per group, a sign generator per element and 2-byte
// stores), 512 x 14336 13.4 -> 12.3 us; 20.8 and 10.6 with the signs applied as
// integers.
template <int E, typename InT, bool ROT, int W>
__global__ __launch_bounds__(64 * W) void xprep_wide_kernel(const InT* __restrict__ x, int64_t batch,
                                                         int64_t in, XSeeds seeds, float rscale,
                                                         _Float16* __restrict__ x16,
                                                         float* __restrict__ xe) {
  constexpr int g = 64 * E;
  // g = 1024 rotates through LDS (half the instructions of the cross-lane form)
  constexpr bool kLds = ROT && E == 16;
  __shared__ __align__(16) float s_rot[kLds ? W : 1][kLds ? kFwht1024Scratch : 4];
  __shared__ uint64_t s_neg[kMaxGroup][E];  // sign bits of 64 elements each
  const int lane = int(threadIdx.x) & 63;
  int wave = int(threadIdx.x) >> 6;
  if constexpr (ROT) wave = __builtin_amdgcn_readfirstlane(wave);
  const int64_t gpr = in / g, ngroups = batch * gpr;
  const int64_t nwaves = int64_t(gridDim.x) * W;
  // the layers of this block's groups: all of them, or one (a row of the grid
  // per layer)
  const int l0 = gridDim.y > 1 ? int(blockIdx.y) : 0;
  const int l1 = gridDim.y > 1 ? l0 + 1 : seeds.nl;
  int64_t grp = int64_t(blockIdx.x) * W + wave;
  const auto row_of = [gpr](int64_t i) HIGGS_INLINE {
    if (ROT && (i >> 32) == 0) return int64_t(uint32_t(i) / uint32_t(gpr));
    return i / gpr;
  };
  // a wave's first weights are on their way while the signs are made
  constexpr bool kVec = E * sizeof(InT) % 16 == 0;
  constexpr int kRaw = kVec ? E * int(sizeof(InT)) / 16 : 1;
  u32x4 raw[kRaw];
  const auto load = [&]() HIGGS_INLINE {
    const int64_t row = row_of(grp);
    const u32x4* src =
        reinterpret_cast<const u32x4*>(x + row * in + (grp - row * gpr) * g + lane * E);
#pragma unroll
    for (int q = 0; q < kRaw; ++q) raw[q] = src[q];
  };
  if constexpr (kVec) {
    if (grp < ngroups) load();
  }
  uint64_t neg[kMaxGroup] = {0, 0, 0, 0};  // of the lane's E elements
  if constexpr (ROT) {
    for (int w = wave; w < (l1 - l0) * E; w += W) {
      const int l = l0 + w / E, q = w % E;
      uint64_t seed = seeds.s[0];
#pragma unroll
      for (int k = 1; k < kMaxGroup; ++k)
        if (l == k) seed = seeds.s[k];
      const uint64_t bits = __ballot(rht_sign_negative(seed, uint32_t(64 * q + lane)));
      if (lane == 0) s_neg[l][q] = bits;
    }
    __syncthreads();
#pragma unroll
    for (int l = 0; l < kMaxGroup; ++l)
      if (l >= l0 && l < l1) neg[l] = s_neg[l][lane * E / 64] >> (lane * E % 64);
  }
  while (grp < ngroups) {
    const int64_t cur = grp;
    const int64_t row = row_of(cur);
    const int64_t kg = (cur - row * gpr) * g;
    const int64_t k0 = kg + lane * E;
    grp += nwaves;
    float u[E];
    if constexpr (kVec) {
#pragma unroll
      for (int q = 0; q < kRaw; ++q) {
        const uint32_t w[4] = {raw[q].x, raw[q].y, raw[q].z, raw[q].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if constexpr (sizeof(InT) == 4) {
            u[4 * q + k] = __uint_as_float(w[k]);
          } else {
            u[8 * q + 2 * k] = __uint_as_float(w[k] << 16);
            u[8 * q + 2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
          }
        }
      }
      if (grp < ngroups) load();
    } else {
      const InT* src = x + row * in + k0;
#pragma unroll
      for (int i = 0; i < E; ++i) {
        if constexpr (sizeof(InT) == 4)
          u[i] = float(src[i]);
        else
          u[i] = __uint_as_float(uint32_t(reinterpret_cast<const uint16_t*>(src)[i]) << 16);
      }
    }
#pragma unroll
    for (int l = 0; l < kMaxGroup; ++l) {
      if (l >= l1) break;  // uniform
      if (l < l0) continue;
      float v[E];
      if constexpr (ROT) {
        // (opaque: kept as they are, not as one 64-lane mask per element, which
        // overflow the scalar registers from g = 1024)
        uint32_t bits[2] = {uint32_t(neg[l]), uint32_t(neg[l] >> 32)};
        asm volatile("" : "+v"(bits[0]), "+v"(bits[1]));
#pragma unroll
        for (int i = 0; i < E; ++i)
          v[i] = __uint_as_float(__float_as_uint(u[i]) ^
                                 ((bits[i / 32] << (31 - i % 32)) & 0x80000000u));
      } else {
#pragma unroll
        for (int i = 0; i < E; ++i) v[i] = u[i];
      }
      if constexpr (ROT) {
        if constexpr (kLds)
          fwht1024_lds(v, s_rot[wave], lane);
        else
          fwht_wave<E>(v, lane, g);
#pragma unroll
        for (int i = 0; i < E; ++i) v[i] *= rscale;
      }
      float m = 0.f;
#pragma unroll
      for (int i = 0; i < E; ++i) m = fmaxf(m, fabsf(v[i]));
      m = wave_max(m, lane);
      const int e = group_exponent(m);
      _Float16* dst = x16 + int64_t(l) * batch * in;
      if constexpr (kLds) {  // lane l holds elements 256 h + 4 l + j in v[4 h + j]
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          uint2 w;
          w.x = pack_h2(ldexpf(v[4 * h], -e), ldexpf(v[4 * h + 1], -e));
          w.y = pack_h2(ldexpf(v[4 * h + 2], -e), ldexpf(v[4 * h + 3], -e));
          *reinterpret_cast<uint2*>(dst + xw_index(batch, in, row, kg + 256 * h + 4 * lane)) = w;
        }
      } else if constexpr (E % 8 == 0) {
#pragma unroll
        for (int q = 0; q < E / 8; ++q) {
          u32x4 w;
          w.x = pack_h2(ldexpf(v[8 * q], -e), ldexpf(v[8 * q + 1], -e));
          w.y = pack_h2(ldexpf(v[8 * q + 2], -e), ldexpf(v[8 * q + 3], -e));
          w.z = pack_h2(ldexpf(v[8 * q + 4], -e), ldexpf(v[8 * q + 5], -e));
          w.w = pack_h2(ldexpf(v[8 * q + 6], -e), ldexpf(v[8 * q + 7], -e));
          *reinterpret_cast<u32x4*>(dst + xw_index(batch, in, row, k0 + 8 * q)) = w;
        }
      } else if constexpr (E > 1) {  // 2 or 4 halves, inside one piece
        uint32_t* p = reinterpret_cast<uint32_t*>(dst + xw_index(batch, in, row, k0));
#pragma unroll
        for (int q = 0; q < E / 2; ++q)
          p[q] = pack_h2(ldexpf(v[2 * q], -e), ldexpf(v[2 * q + 1], -e));
      } else {
        dst[xw_index(batch, in, row, k0)] = static_cast<_Float16>(ldexpf(v[0], -e));
      }
      if (lane == 0) xe[int64_t(l) * ngroups + cur] = ldexpf(1.0f, e);
    }
  }
}

// The same with one group per block of four waves (g = 256 E): a wave's serial
// chain of loads, butterflies and stores is a quarter as long, and 64 elements
// per lane took all of a wave's registers. Thread t holds elements
// [tE, (t + 1)E); butterflies over the top two element bits go through LDS. The
// stages run in the same order and each is (a + b, a - b): the same values bit
// for bit. Block b takes group grp0 + b of layer blockIdx.y (one group: with a
// loop over groups the signs move out of it, into more registers than there
// are). Whole calls of 256 outputs against a wave per group, 4096 weights per
// row: g = 4096 23.3 -> 18.5 us at 65 rows, 44 -> 36 at 2048 (fp32); g = 2048
// 22.1 -> 19.4 at 200 rows, 36.8 -> 37.3 at 2048; g = 1024 19.0 -> 18.5 at 65
// rows, 31 -> 37 at 2048.
template <int E, typename InT, bool ROT>
__global__ __launch_bounds__(256) void xprep_wide4_kernel(const InT* __restrict__ x, int64_t batch,
                                                          int64_t in, int64_t grp0, XSeeds seeds,
                                                          float rscale,
                                                          _Float16* __restrict__ x16,
                                                          float* __restrict__ xe) {
  constexpr int g = 256 * E;
  __shared__ float s_v[2][ROT ? g : 1];
  __shared__ float s_m[4];
  const int tid = int(threadIdx.x), lane = tid & 63, wave = tid >> 6;
  const int64_t gpr = in / g, grp = grp0 + blockIdx.x;
  const int64_t row = uint32_t(grp) / uint32_t(gpr);
  const int64_t k0 = (grp - row * gpr) * g + tid * E;
  float v[E];
  const InT* src = x + row * in + k0;
  if constexpr (sizeof(InT) == 4) {
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
      const f32x4 u = reinterpret_cast<const f32x4*>(src)[q];
      v[4 * q] = u.x; v[4 * q + 1] = u.y; v[4 * q + 2] = u.z; v[4 * q + 3] = u.w;
    }
  } else {
#pragma unroll
    for (int q = 0; q < E / 4; ++q) {
      const uint2 u = reinterpret_cast<const uint2*>(src)[q];
      v[4 * q] = __uint_as_float(u.x << 16);
      v[4 * q + 1] = __uint_as_float(u.x & 0xffff0000u);
      v[4 * q + 2] = __uint_as_float(u.y << 16);
      v[4 * q + 3] = __uint_as_float(u.y & 0xffff0000u);
    }
  }
  const int64_t layer = blockIdx.y;
  if constexpr (ROT) {
    uint64_t seed = seeds.s[0];
#pragma unroll
    for (int l = 1; l < kMaxGroup; ++l)
      if (layer == l) seed = seeds.s[l];
#pragma unroll
    for (int i = 0; i < E; ++i)
      if (rht_sign_negative(seed, uint32_t(tid * E + i))) v[i] = -v[i];
    fwht_in_lane<E>(v);
    fwht_cross_lane<E>(v, lane, 64 * E);
    // wave bits 0 and 1: the lower wave of a pair keeps a + b, the upper one
    // a - b (a the lower wave's value)
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const int bit = 1 << st;
      float* buf = s_v[st];
#pragma unroll
      for (int i = 0; i < E; ++i) buf[tid * E + i] = v[i];
      __syncthreads();
      const float* o = buf + (tid ^ (64 * bit)) * E;
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = (wave & bit) ? o[i] - v[i] : v[i] + o[i];
    }
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] *= rscale;
  }
  float m = 0.f;
#pragma unroll
  for (int i = 0; i < E; ++i) m = fmaxf(m, fabsf(v[i]));
  m = wave_max(m, lane);
  if (lane == 0) s_m[wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
  const int e = group_exponent(m);
  _Float16* dst = x16 + layer * batch * in;
#pragma unroll
  for (int q = 0; q < E / 4; ++q) {
    uint2 w;
    w.x = pack_h2(ldexpf(v[4 * q], -e), ldexpf(v[4 * q + 1], -e));
    w.y = pack_h2(ldexpf(v[4 * q + 2], -e), ldexpf(v[4 * q + 3], -e));
    *reinterpret_cast<uint2*>(dst + xw_index(batch, in, row, k0 + 4 * q)) = w;
  }
  if (tid == 0) xe[layer * batch * gpr + grp] = ldexpf(1.0f, e);
}

// ---------------------------------------------------------------------------
// The product.
// ---------------------------------------------------------------------------
// The weights of K that K-group q of a block takes, the block's split covering
// [split kps, split kps + kps) of them: equal parts (rounded up to 128) in turn,
// so group 0 has the most stages of 64, and every group waits for as many (two
// if group 0 has one). A group without stages still requests one of the row's,
// which it does not use.
struct WideRange {
  int first;   // first weight
  int stages;  // stages of the group
  int turns;   // stages to wait for
};

__host__ __device__ inline WideRange wide_range(int in, int kps, int split, int groups, int q) {
  const int kbeg = split * kps, kend = kbeg + kps < in ? kbeg + kps : in;
  const int part = groups == 1 ? kend - kbeg
                               : (kend - kbeg + 128 * groups - 1) / (128 * groups) * 128;
  const int first = kbeg + q * part < kend ? kbeg + q * part : kend;
  const int end = first + part < kend ? first + part : kend;
  return WideRange{first < in - 64 ? first : in - 64, (end - first) >> 6, part >> 6};
}

// One launch covers nl layers (1..kMaxGroup) that read the same activations.
// Work items are numbered layer by layer, row tile by row tile, then by
// K-split, then by column tile. Consecutive layers with items of one length
// form a run; XCD x (blocks are dealt to the XCDs round robin) takes the x-th
// eighth of each run, so that the column tiles that decode the same codes, and
// neighbouring row tiles, which read the same activations, run on one XCD and
// meet in its L2, and every XCD has its part of the longest items, which come
// first. (With eighths of all items together some XCDs had only long ones:
// 8192, 1024 and 1024 rows x 8192, 10-bit codes, g = 128, 257 batch rows 410 us,
// 176 now, 250 in 64-column launches; with every layer dealt by itself each
// XCD reads every layer's copy of the activations: four layers of 512 x 1024 at
// 700 rows 28.9 -> 31.4 us.)
struct QW {
  const _Float16* x16;  // copy c: + c * x16_stride
  const float* xe;      // [batch][gpr] powers of two (copy c: + c * xe_stride)
  int64_t x16_stride, xe_stride;
  const float* grid;
  int batch, pair_table, log2g, in, gpr, nl, ctiles;
  int item0[kMaxGroup];   // layer l's first work item
  int run0[kMaxGroup];    // its run's first work item
  int run[kMaxGroup];     // its run's number of work items
  int turn0[kMaxGroup];   // blocks per XCD before its run's first
  int xcopy[kMaxGroup];   // the layer's copy of the activations
  int kps[kMaxGroup];     // weights of K per split (a multiple of 256)
  int splits[kMaxGroup];
  int out[kMaxGroup];
  const uint8_t* codes[kMaxGroup];
  const uint16_t* scales[kMaxGroup];
  float* dst[kMaxGroup];  // [splits][batch][out]
};

// Waits until at most N of this wave's vector memory operations and none of
// its LDS operations are outstanding.
template <int N>
__device__ inline void wait_loads() {
  static_assert(N >= 0 && N < 64, "the counter has six bits");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

// G64: groups of 64 weights, which end at every stage; larger groups end at
// even stages only (K-ranges start at multiples of 128, and such rows have an
// even number of stages).
template <int BITS, int NB, int CW, int KG, int kWaves, bool G64>
__global__ __launch_bounds__(64 * kWaves, kWaves / 4) void qgemm_wide_kernel(const QW a) {
  using F = GFmt<BITS>;
  constexpr int kThreads = 64 * kWaves;
  constexpr int kW = F::kWords;
  // 256-byte entry slots hold 32 copies in their low halves; the high halves
  // of 16 slots hold the waves' row factors (rows_of below). 10-bit codes: 16
  // copies, no such space.
  constexpr int kCopies = F::kRL < 5 ? 1 << F::kRL : 32;
  constexpr bool kRowLds = F::kStride == 8;
  constexpr int kEntries = BITS == 16 ? 256 : 1 << BITS;
  constexpr int kEntryU4 = (1 << F::kStride) / 16;
  constexpr int kLutU4 = kEntries * kEntryU4;
  constexpr int kCols = 32 * NB * CW;       // CW waves side by side
  constexpr int kRows = 64 * kWaves / (CW * KG);
  constexpr int kGWaves = kWaves / KG;  // waves of a K-group
  constexpr int kDma = kCols / 8 / kGWaves;  // activation loads per wave and stage
  constexpr int kStageBytes = kCols * 128;  // 64 weights of kCols batch rows
  constexpr bool kPair = BITS != 16;        // codes requested for two stages at a time
  // code loads per stage: one per row set, two for 10- and 16-bit pairs
  constexpr int kLoads = BITS >= 10 ? 4 : 2;
  // LDS reads and address instructions per product that feed the next step
  constexpr int kStepReads = NB + (BITS == 16 ? 16 : 8);
  constexpr int kReads = (kStepReads + 2 * NB - 1) / (2 * NB);
  constexpr int kValu = BITS == 8 ? kReads : 2 * kReads;
  __shared__ u32x4 s_mem[kLutU4 + KG * kBufs * kStageBytes / 16];
  const char* const s_lut = reinterpret_cast<const char*>(s_mem);

  const int tid = int(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kgrp = wave / kGWaves, gwave = wave % kGWaves;
  const int rw = gwave % (kRows / 64), cw = gwave / (kRows / 64);
  char* const s_x0 = reinterpret_cast<char*>(s_mem + kLutU4);
  char* const s_x = s_x0 + kgrp * kBufs * kStageBytes;  // the K-group's stages
  const int ahalf = lane >> 5;

  // ---- work item ----
  const int xcd = int(blockIdx.x) % 8, turn = int(blockIdx.x) / 8;
  int run0 = 0, run = a.run[0], turn0 = 0;
#pragma unroll
  for (int l = 1; l < kMaxGroup; ++l)
    if (l < a.nl && turn >= a.turn0[l]) {
      run0 = a.run0[l];
      run = a.run[l];
      turn0 = a.turn0[l];
    }
  const int per = run / 8, rem = run % 8;
  if (turn - turn0 >= per + int(xcd < rem)) return;  // the run's last turn is not full
  const int item = run0 + xcd * per + min(xcd, rem) + turn - turn0;
  int L = 0;
#pragma unroll
  for (int l = 1; l < kMaxGroup; ++l)
    if (l < a.nl && item >= a.item0[l]) L = l;
  const uint8_t* codes = a.codes[0];
  const uint16_t* scales = a.scales[0];
  float* dst = a.dst[0];
  int out = a.out[0], item0 = 0, kps = a.kps[0], splits = a.splits[0], xcopy = a.xcopy[0];
#pragma unroll
  for (int l = 1; l < kMaxGroup; ++l)
    if (L == l) {
      codes = a.codes[l];
      scales = a.scales[l];
      dst = a.dst[l];
      out = a.out[l];
      item0 = a.item0[l];
      kps = a.kps[l];
      splits = a.splits[l];
      xcopy = a.xcopy[l];
    }
  const int in = a.in, gpr = a.gpr, log2g = a.log2g, batch = a.batch;
  // (uniform, but divided in vector registers: read back to scalar ones)
  const int wl = item - item0;
  const int wt = __builtin_amdgcn_readfirstlane(wl / a.ctiles);
  const int ctile = wl - wt * a.ctiles;
  const int rtile = __builtin_amdgcn_readfirstlane(wt / splits);
  const int split = wt - rtile * splits;
  const int row0 = rtile * kRows + rw * 64;  // the wave's first row
  const int col0 = ctile * kCols;                             // the block's first batch row
  // the K-group's part of the block's K-range
  const WideRange range = wide_range(in, kps, split, KG, kgrp);
  const int kbeg = range.first;
  const int nmax = range.turns;
  const int nst = range.stages;        // stages (K-blocks of 64 weights)
  const int last = max(nst - 1, 0);    // stage that requests past the end repeat
  dst += int64_t(split) * batch * out;

  // ---- activations of a stage: memory to LDS, 1 KiB (8 batch rows) per wave
  //      instruction; rows past the batch repeat the chunk's last row (their
  //      columns are never stored) ----
  const int chunk = col0 / kChunk;
  const int crows = min(kChunk, batch - chunk * kChunk);
  const __amdgpu_buffer_rsrc_t xrs =
      rsrc(a.x16 + int64_t(xcopy) * a.x16_stride + int64_t(chunk) * kChunk * in,
           uint32_t(crows) * uint32_t(in) * 2u);
  uint32_t xoff[kDma];
#pragma unroll
  for (int i = 0; i < kDma; ++i) {
    const int r = col0 - chunk * kChunk + (i * kGWaves + gwave) * 8 + (lane >> 3);
    xoff[i] = uint32_t(min(r, crows - 1)) * 128u + uint32_t(lane & 7) * 16u;
  }
  const uint32_t stage_stride = uint32_t(crows) * 128u;
  auto issue_x = [&](int st, int buf) HIGGS_INLINE {
    const uint32_t soff = uint32_t((kbeg >> 6) + min(st, last)) * stage_stride;
#pragma unroll
    for (int i = 0; i < kDma; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          xrs, (lds_void*)(s_x + buf * kStageBytes + (i * kGWaves + gwave) * 1024), 16,
          int(xoff[i]), int(soff), 0, 0);
  };

  // ---- codes: lane l of row set m holds half l / 32 (32 weights) of each
  //      K-block of row 32 m + l % 32 ----
  constexpr uint32_t kKBBytes = 8 * kW;
  const uint32_t row_bytes = uint32_t(in >> 6) * kKBBytes;
  const __amdgpu_buffer_rsrc_t crs = rsrc(codes, uint32_t(out) * row_bytes);
  uint32_t cbase[2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
    cbase[m] = uint32_t(min(row0 + 32 * m + (lane & 31), out - 1)) * row_bytes +
               uint32_t(kbeg >> 6) * kKBBytes + 4u * kW * uint32_t(ahalf);
  auto fetch = [&](int st, uint32_t (&d)[2][kW]) HIGGS_INLINE {
    const uint32_t off = kKBBytes * uint32_t(min(st, last));
#pragma unroll
    for (int m = 0; m < 2; ++m) load_codes<BITS>(crs, cbase[m] + off, d[m]);
  };

  // ---- scales of a group: lane l -> row row0 + l; its columns' exponents ----
  const __amdgpu_buffer_rsrc_t srs = rsrc(scales, uint32_t(out) * uint32_t(gpr) * 2u);
  const uint32_t srow = uint32_t(min(row0 + lane, out - 1)) * uint32_t(gpr);
  const float* xe = a.xe + int64_t(xcopy) * a.xe_stride;
  const float* xep[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t)
    xep[t] = xe + int64_t(min(col0 + cw * 32 * NB + 32 * t + (lane & 31), batch - 1)) * gpr;
  auto load_units = [&](int grp, float& s, float (&xs)[NB]) HIGGS_INLINE {
    grp = min(grp, gpr - 1);
    const uint16_t h = uint16_t(
        __builtin_amdgcn_raw_buffer_load_b16(srs, int((srow + uint32_t(grp)) * 2u), 0, 0));
    s = float(__builtin_bit_cast(_Float16, h));
#pragma unroll
    for (int t = 0; t < NB; ++t) xs[t] = xep[t][grp];
  };

  // the stages' loads are issued one stage after the other: the waits below
  // count on that order
  uint32_t cod0[2][kW], cod1[2][kW];
  fetch(0, cod0);
  if constexpr (kPair) fetch(1, cod1);
  __builtin_amdgcn_sched_barrier(0);
  issue_x(0, 0);
  __builtin_amdgcn_sched_barrier(0);
  issue_x(1, 1);
  __builtin_amdgcn_sched_barrier(0);
  issue_x(2, 2);
  __builtin_amdgcn_sched_barrier(0);
  int grp = kbeg >> log2g;
  float s_cur, s_nxt, x_cur[NB], x_nxt[NB];
  load_units(grp, s_cur, x_cur);
  load_units(grp + 1, s_nxt, x_nxt);

  // ---- the table: kCopies copies of each entry, whole 16-byte words ----
  {
    constexpr int kPer = kCopies / 4;  // words per entry
    for (int n = tid; n < kEntries * kPer; n += kThreads) {
      const int e = n / kPer;
      float gx, gy = 0.f;
      if constexpr (BITS == 16) {
        gx = a.grid[e];
      } else {
        gx = a.pair_table ? a.grid[e & 15] : a.grid[2 * e];
        gy = a.pair_table ? a.grid[e >> 4] : a.grid[2 * e + 1];
      }
      const uint32_t v = pack_h2(gx, gy);
      s_mem[e * kEntryU4 + n % kPer] = u32x4{v, v, v, v};
    }
  }
  const uint32_t copy_off = uint32_t(lane & (kCopies - 1)) << 2;

  f16x_acc acc[2][NB];    // sums of the current scale group
  f16x_acc total[2][NB];  // scaled sums of the groups before it
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int t = 0; t < NB; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][t][r] = total[m][t][r] = 0.f;

  // B operand of step s, tile t: piece 4 ahalf + s of column 32 t + l % 32
  const int bcol = (cw * 32 * NB + (lane & 31)) * 128;
  uint32_t bpos[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) bpos[s] = uint32_t(bcol + (((4 * ahalf + s) ^ (lane & 7)) << 4));

  int buf = 0;  // the current stage's buffer

  // ---- a stage: 4 steps of 16 weights per K-half, each 2 NB products. The
  //      operands of a step are read from LDS while the step before it
  //      multiplies; step 3 reads the next stage's first operands. ----
  struct Step {
    half8 a[2];
    half8 b[NB];
  };
  Step ops[2];
  auto load_step = [&](int buf, const uint32_t (&cod)[2][kW], int s, Step& o) HIGGS_INLINE {
    const char* xb = s_x + buf * kStageBytes;
#pragma unroll
    for (int t = 0; t < NB; ++t)
      o.b[t] = *reinterpret_cast<const half8*>(xb + bpos[s] + t * 4096);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      uint32_t a32[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (BITS == 16) {
          const int cc = 4 * s + q;
          const uint32_t o0 = lut_off_byte<kW>(cod[m], 2 * cc, copy_off);
          const uint32_t o1 = lut_off_byte<kW>(cod[m], 2 * cc + 1, copy_off);
          a32[q] = uint32_t(*reinterpret_cast<const uint16_t*>(s_lut + o0)) |
                   (uint32_t(*reinterpret_cast<const uint16_t*>(s_lut + o1)) << 16);
        } else {
          a32[q] = *reinterpret_cast<const uint32_t*>(s_lut +
                                                      lut_off<BITS>(cod[m], 4 * s + q, copy_off));
        }
      }
      o.a[m] = __builtin_bit_cast(half8, u32x4{a32[0], a32[1], a32[2], a32[3]});
    }
  };
  auto mul_step = [&](const Step& o) HIGGS_INLINE {
#pragma unroll
    for (int t = 0; t < NB; ++t)
#pragma unroll
      for (int m = 0; m < 2; ++m)
        acc[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o.a[m], o.b[t], acc[m][t], 0, 0, 0);
    // the next step's LDS reads between the products
#pragma unroll
    for (int i = 0; i < 2 * NB; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one product
      __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, kReads, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // One stage (codes `cod`, buffer `buf`), then the first operands of the next
  // one (codes `cnext`, buffer `bnext`). kLate: loads issued after those of
  // stage st + 2 by the time of its wait (see below).
  auto stage = [&](int st, const uint32_t (&cod)[2][kW], const uint32_t (&cnext)[2][kW],
                   auto LATE) HIGGS_INLINE {
    const int bnext = buf + 1 == kBufs ? 0 : buf + 1;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      load_step(buf, cod, s + 1, ops[(s + 1) & 1]);
      mul_step(ops[s & 1]);
    }
    // Step 3's operands are in registers: this stage's buffer is free once
    // every wave is here. Loads are counted in order: after stage st + 1's
    // (issued two stages ago) came at least the kDma loads of stage st + 2 and
    // kLate code loads, so waiting for all but those waits for stage st + 1.
    constexpr int kWait = kDma + decltype(LATE)::value;
    __builtin_amdgcn_sched_barrier(0);
    wait_loads<kWait>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    issue_x(st + 3, buf);
    load_step(bnext, cnext, 0, ops[0]);
    mul_step(ops[1]);
    buf = bnext;
  };
  // Factor f of the lane's row (lane l: row l of the wave's 64) for the rows
  // that the lane's accumulators hold: put_rows, then row_quad(m, q) gives
  // those of rows 32 m + 8 q + 4 ahalf + 0..3.
  char* const s_rows = reinterpret_cast<char*>(s_mem) + wave * 512 + 128;
  float row_f = 0.f;
  int half4 = 0;
  auto put_rows = [&](float f) HIGGS_INLINE {
    half4 = 4 * ahalf;  // opaque: addresses are formed here, not kept in registers
    asm volatile("" : "+v"(half4));
    row_f = f;
    if constexpr (kRowLds) {
      wave_lds_sync();
      *reinterpret_cast<float*>(s_rows + ahalf * 256 + (lane & 31) * 4) = f;
      wave_lds_sync();
    }
  };
  auto row_quad = [&](int m, int q, float (&f)[4]) HIGGS_INLINE {
    if constexpr (kRowLds) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(s_rows + m * 256 + 32 * q + 4 * half4);
      f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) f[k] = __shfl(row_f, 32 * m + 8 * q + half4 + k, 64);
    }
  };
  // Adds the group's sums, in units of the row's scale times the column's power
  // of two, to the totals: one rounding (the power of two is exact).
  auto add_totals = [&]() HIGGS_INLINE {
    put_rows(s_cur);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float f[4];
        row_quad(m, q, f);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
          for (int t = 0; t < NB; ++t) {
            const int r = 4 * q + k;
            total[m][t][r] = fmaf(acc[m][t][r] * x_cur[t], f[k], total[m][t][r]);
            acc[m][t][r] = 0.f;
          }
      }
  };
  // after stage st: at the end of a scale group inside the block's K-range
  auto end_group = [&](int st) HIGGS_INLINE {
    const int gn = (kbeg + (st + 1) * 64) >> log2g;
    if (st + 1 < nst && gn != grp) {
      add_totals();
      s_cur = s_nxt;
#pragma unroll
      for (int t = 0; t < NB; ++t) x_cur[t] = x_nxt[t];
      grp = gn;
      load_units(grp + 1, s_nxt, x_nxt);
    }
  };
  // stage 0 is there, in every wave's part of it; so is the table
  __builtin_amdgcn_sched_barrier(0);
  wait_loads<2 * kDma>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  load_step(0, cod0, 0, ops[0]);

  // Two stages per turn. Codes of pairs of K-blocks (64 bytes of a row for
  // 8-bit codes) are requested together, two stages ahead; scalar 8-bit codes
  // (64 bytes per K-block) one stage ahead.
  constexpr int kLate = kPair ? 2 * kLoads : kLoads;
  // a stage past the K-group's range, for the barriers of the other group
  auto idle = [&]() HIGGS_INLINE {
    if constexpr (KG > 1) {
      wait_loads<0>();
      __builtin_amdgcn_s_barrier();
    }
  };
  for (int st = 0; st < nmax; st += 2) {
    if (KG > 1 && st >= nst) {
      idle();
      idle();
      continue;
    }
    if constexpr (kPair) {
      uint32_t nxt0[2][kW], nxt1[2][kW];
      fetch(st + 2, nxt0);
      fetch(st + 3, nxt1);
      __builtin_amdgcn_sched_barrier(0);
      stage(st, cod0, cod1, std::integral_constant<int, kLate>{});
      if constexpr (G64) end_group(st);
      if (!G64 || st + 1 < nst) {
        stage(st + 1, cod1, nxt0, std::integral_constant<int, 0>{});
        end_group(st + 1);
      } else {
        idle();
      }
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int w = 0; w < kW; ++w) {
          cod0[m][w] = nxt0[m][w];
          cod1[m][w] = nxt1[m][w];
        }
    } else {
      fetch(st + 1, cod1);
      __builtin_amdgcn_sched_barrier(0);
      stage(st, cod0, cod1, std::integral_constant<int, kLate>{});
      if constexpr (G64) end_group(st);
      if (!G64 || st + 1 < nst) {
        fetch(st + 2, cod0);
        __builtin_amdgcn_sched_barrier(0);
        stage(st + 1, cod1, cod0, std::integral_constant<int, kLate>{});
        end_group(st + 1);
      } else {
        idle();
      }
    }
  }
  if (KG == 1 || nst > 0) add_totals();

  // No load may be on its way into LDS when a wave leaves or reuses a buffer.
  wait_loads<0>();
  __syncthreads();
  // ---- store through LDS (the activation buffers are free) so that lanes
  //      write consecutive rows: 32 x 32 tiles; with several K-groups, group 0
  //      adds the others' sums for the same rows and columns, in turn ----
  constexpr int kORow = 33;                // floats per staged column
  constexpr int kOTile = 32 * kORow;
  constexpr int kOTiles = KG == 1 ? 1 : NB;  // tiles per wave at a time
  static_assert(kWaves * kOTiles * kOTile * 4 <= KG * kBufs * kStageBytes, "output staging fits");
  float* s_o = reinterpret_cast<float*>(s_x0) + wave * kOTiles * kOTile;
  // value of wave tile (m, t) into the wave's tile buffer o
  auto put_tile = [&](int m, int t, float* o) HIGGS_INLINE {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rl = 8 * (r / 4) + 4 * ahalf + (r % 4);
      o[(lane & 31) * kORow + rl] = total[m][t][r];
    }
  };
  auto store_tile = [&](int m, int t, const float* o) HIGGS_INLINE {
    const int row = row0 + 32 * m + (lane & 31);
    const int colt = col0 + cw * 32 * NB + 32 * t;
    const __amdgpu_buffer_rsrc_t drs = rsrc(dst + int64_t(colt) * out, 0x7fffffffu);
    // batch rows of this half of the wave that are stored (none past out)
    const int nc = row < out ? batch - colt - ahalf : 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int c = 2 * i + ahalf;
      float v = o[c * kORow + (lane & 31)];
#pragma unroll
      for (int q = 1; q < KG; ++q)
        v += o[q * kGWaves * kOTiles * kOTile + c * kORow + (lane & 31)];
      const uint32_t off = (uint32_t(c) * uint32_t(out) + uint32_t(row)) * 4u;
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), drs,
                                            int(2 * i < nc ? off : kOffNone), 0, 0);
    }
  };
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    if constexpr (KG > 1) {
#pragma unroll
      for (int t = 0; t < NB; ++t) put_tile(m, t, s_o + t * kOTile);
      __syncthreads();
      if (kgrp == 0) {
#pragma unroll
        for (int t = 0; t < NB; ++t) store_tile(m, t, s_o + t * kOTile);
      }
      __syncthreads();
    } else {
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        wave_lds_sync();
        put_tile(m, t, s_o);
        wave_lds_sync();
        store_tile(m, t, s_o);
      }
    }
  }
}

int64_t align256(int64_t v) { return (v + 255) / 256 * 256; }

int pair_bits(int p, int n) { return p == 1 ? 2 * code_bits(p, n) : code_bits(p, n); }

// Block shapes: rows x batch columns, and the waves' arrangement; times in us
// measured on MI355X for 8-bit codes: a stage of 64 weights of K with few
// blocks running and with one on every compute unit (clocks and L2 shared),
// and the fold of a scale group into the totals.
struct WShape {
  int rows, cols;
  double stage_few, stage_full, unit;
};
constexpr int kShapes = 4;
constexpr WShape kShape[kShapes] = {
    {256, 128, 0.62, 0.93, 1.2},   // one K-group of 4 waves, 64 x 128 each
    {256, 128, 0.77, 1.06, 0.7},   // one K-group of 8 waves, 64 x 64 each
    {128, 128, 0.42, 0.58, 0.4},   // two K-groups of 4 waves, 64 x 64 each
    {128, 64, 0.26, 0.36, 0.20},   // four K-groups of 2 waves, 64 x 64 each
};

// A layer's block shape and K-split.
struct WPlan {
  int shape;
  int64_t kps, splits;
};

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The shape and split with the least modelled time: rounds of one block per
// compute unit, each a start and end (5 us) and its stages; a split adds the
// reduction launch, its round trips and the partial sums' traffic. Large tiles
// decode a code for more columns and read less; small ones, and splits, fill
// the chip when the layer or the batch is small. The plan depends on the sizes
// only. Where the 64-column product's workspace fits in the library's fixed
// scratch, so does the plan's (unsplit if need be): the calls that use it take
// what they took with that product. Elsewhere the partial sums take what
// they need (128 x 131072, 129 rows: 819 us unsplit, 45 with 128 splits, 83
// in 64-column launches).
WPlan plan_wide(int64_t batch, int64_t out, int64_t in, int g, int bits) {
  constexpr int kSplits[] = {1,  2,  3,  4,  5,  6,  7,  8,  10, 12,  14,
                             16, 19, 24, 28, 32, 48, 56, 64, 96, 128, 256};
  const int64_t x_bytes = align256(batch * in * 2) + align256(batch * (in / g) * 4);
  // measured stage times of the other code widths against 8-bit codes
  const double width = bits == 8 ? 1.0 : bits == 6 ? 1.08 : bits == 10 ? 1.5 : 1.3;
  // The 256-row shape: from g = 256 the one that decodes a code for twice the
  // columns, below it the one whose folds, two or one stage apart, cost less
  // (28672 x 4096 at 2048 rows: g = 1024 504 us against 531, 256: 593 and 588,
  // scalar 16 points with g = 128: 705 and 648); 10-bit codes, whose decoding
  // costs most, take the first at g = 128 as well (and g = 64 is scalar).
  const int large = g < 256 && bits != 10 ? 1 : 0;
  const int first = batch <= 64 ? 3 : large, last = batch <= 64 ? 3 : 2;
  WPlan best{first, ceil_div(in, 256) * 256, 1};
  double best_t = 1e30;
  for (int sh = first; sh <= last; sh += 2 - large) {
    const WShape& S = kShape[sh];
    const int64_t blocks = ceil_div(out, S.rows) * ceil_div(batch, S.cols);
    int64_t last_kps = 0;
    for (const int want : kSplits) {
      const int64_t kps = ceil_div(ceil_div(in, want), 256) * 256;
      if (kps == last_kps) continue;
      last_kps = kps;
      const int64_t s = ceil_div(in, kps);
      if (s > 1 && x_bytes + align256(s * batch * out * 4) > kScratchBytes &&
          qgemm64_workspace_bytes(batch, out, in, g, bits) <= kScratchBytes)
        break;
      const double used = std::min(1.0, double(blocks * s) / 256.0);
      const double stage = (S.stage_few + (S.stage_full - S.stage_few) * used) * width;
      const double t = double(ceil_div(blocks * s, 256)) *
                           (double(kps) / 64 * stage + double(kps) / g * S.unit + 5.0) +
                       (s > 1 ? 4.0 + 0.09 * double(s) + double((2 * s + 1) * batch * out) * 1e-6
                              : 0.0);
      if (t < best_t * 0.97) {
        best_t = t;
        best = WPlan{sh, kps, s};
      }
    }
  }
  return best;
}

struct WLayout {
  int64_t x16, xe, part[kMaxGroup], total;
};

WLayout wide_layout(int64_t batch, const int64_t* outs, int nl, int nx, int64_t in, int g,
                    int bits) {
  WLayout L;
  L.x16 = 0;
  L.xe = align256(nx * batch * in * 2);
  int64_t at = L.xe + align256(nx * batch * (in / g) * 4);
  for (int l = 0; l < nl; ++l) {
    const WPlan sp = plan_wide(batch, outs[l], in, g, bits);
    L.part[l] = at;
    if (sp.splits > 1) at += align256(sp.splits * batch * outs[l] * 4);
  }
  L.total = at;
  return L;
}

template <typename InT, bool ROT>
hipError_t launch_xprep_wide(const InT* x, int64_t batch, int64_t in, int g, const XSeeds& seeds,
                             _Float16* x16, float* xe, hipStream_t stream) {
  const float rscale = float(1.0 / std::sqrt(double(g)));
  const int64_t groups = batch * (in / g);
  // a block per group (xprep_wide4_kernel): g = 4096 always; g = 2048 where a
  // wave per group would be few waves
  if (g == 4096 || (g == 2048 && groups * seeds.nl <= 1400)) {
    constexpr int64_t kMost = 1 << 23;  // blocks of a launch: below 2^32 threads
    for (int64_t g0 = 0; g0 < groups; g0 += kMost) {
      const dim3 grid{unsigned(std::min(kMost, groups - g0)), unsigned(seeds.nl)}, block{256};
      if (g == 2048)
        hipLaunchKernelGGL((xprep_wide4_kernel<8, InT, ROT>), grid, block, 0, stream, x, batch,
                           in, g0, seeds, rscale, x16, xe);
      else
        hipLaunchKernelGGL((xprep_wide4_kernel<16, InT, ROT>), grid, block, 0, stream, x, batch,
                           in, g0, seeds, rscale, x16, xe);
    }
    return hipGetLastError();
  }
  // 16 waves share a block's signs where that leaves a block for every compute
  // unit, i.e. from 4096 groups; four below (600 groups in blocks of 16 would
  // use 38 compute units) and where there are no signs (5.2 us either way at
  // 300 x 5120)
  const bool big = ROT && g <= 1024 && groups >= 4096;
  const int w = big ? 16 : 4;
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((groups + w - 1) / w, 8192 / w));
  // few groups: a wave makes one layer's copy of its groups, not all of them
  const unsigned rows = big ? 1 : unsigned(seeds.nl);
  switch (g) {
#define HIGGS_XPREP(G)                                                                         \
  case G:                                                                                      \
    if (big)                                                                                   \
      hipLaunchKernelGGL((xprep_wide_kernel<G / 64, InT, ROT, ROT && G <= 1024 ? 16 : 4>),     \
                         dim3(unsigned(blocks), rows), dim3(1024), 0, stream, x, batch, in,    \
                         seeds, rscale, x16, xe);                                                     \
    else                                                                                       \
      hipLaunchKernelGGL((xprep_wide_kernel<G / 64, InT, ROT, 4>),                             \
                         dim3(unsigned(blocks), rows), dim3(256), 0, stream, x, batch, in,     \
                         seeds, rscale, x16, xe);                                              \
    return hipGetLastError();
    HIGGS_XPREP(64)
    HIGGS_XPREP(128)
    HIGGS_XPREP(256)
    HIGGS_XPREP(512)
    HIGGS_XPREP(1024)
    HIGGS_XPREP(2048)
#undef HIGGS_XPREP
    default:
      return hipErrorInvalidValue;
  }
}

template <int BITS, int NB, int CW, int KG, int W, bool G64>
hipError_t launch_shape(const QW& a, unsigned blocks, hipStream_t stream) {
  hipLaunchKernelGGL((qgemm_wide_kernel<BITS, NB, CW, KG, W, G64>), dim3(blocks),
                     dim3(64 * W), 0, stream, a);
  return hipGetLastError();
}

// The shapes that plan_wide gives a code width and group size (g = 64 exists
// for scalar grids only; up to 64 rows, shape 3, so do the calls).
template <int BITS>
hipError_t launch_bits(const QW& a, int shape, unsigned blocks, hipStream_t stream) {
  constexpr bool kScalar = BITS == 8 || BITS == 16;
  if (a.log2g == 6) {
    if constexpr (kScalar) {
      if (shape == 1) return launch_shape<BITS, 2, 2, 1, 8, true>(a, blocks, stream);
      if (shape == 2) return launch_shape<BITS, 2, 2, 2, 8, true>(a, blocks, stream);
      if (shape == 3) return launch_shape<BITS, 2, 1, 4, 8, true>(a, blocks, stream);
    }
    return hipErrorInvalidValue;
  }
  if (shape == 0) return launch_shape<BITS, 4, 1, 1, 4, false>(a, blocks, stream);
  if (shape == 2) return launch_shape<BITS, 2, 2, 2, 8, false>(a, blocks, stream);
  if constexpr (BITS != 10)
    if (shape == 1) return launch_shape<BITS, 2, 2, 1, 8, false>(a, blocks, stream);
  if constexpr (BITS == 16)
    if (shape == 3) return launch_shape<BITS, 2, 1, 4, 8, false>(a, blocks, stream);
  return hipErrorInvalidValue;
}

}  // namespace

// From 65 rows the wide blocks are the faster ones for single layers (65 rows:
// 4096 x 4096 25 -> 23 us, 14336 x 4096 46 -> 34; 129 rows: 39 -> 27, 72 -> 42)
// but for a few (28672 x 8192, 10-bit codes, g = 128: 214 us against 243 at 129
// rows). Calls of two layers of 14336 x 4096 lose at 65 and 80 rows (50 us
// against 57, 53 against 58), with 10-bit codes up to 160 (129 rows: 100 against
// 118; g = 128, 257 rows: 220 against 254): each layer has the K-split of a single call, whose result it has
// to match bit for bit, and whose blocks fill the chip alone. Plans that weigh
// such a pair in made it 44 us at 80 rows, and single layers of 65 to 512 rows
// up to 35% slower. Up to 64 rows those are as fast or faster (64 rows, 4096 x
// 14336, 256 points: 28 us against 34) except where their folds of many small
// groups or two lookups per pair weigh: g = 64 (64 rows, 4096 x 14336: 16 points
// 82 -> 38, 256 scalar points 167 -> 42; 32 rows, 14336 x 4096: 65 -> 32, 89 ->
// 36; 4096 x 4096, 16 points: 21.5 against 21.2 at 32 rows and less than that
// at 16) and scalar 256-point grids with g = 128 (64 rows: 68 -> 37, 64 -> 35;
// 32 rows: 30 against 34). On long rows a layer of few outputs loses at small
// batches (600 x 14336, 16 points: 20 us against 24 at 17 rows, 32 against 30
// at 64), so the lines lie higher there. The limits on `in` keep byte offsets within 32 bits
// and rows worth splitting.
bool use_qgemm_wide(int64_t batch, int64_t in, int p, int n, int g) {
  if (batch >= (int64_t(1) << 24) || in < 512 || in > (int64_t(1) << 20)) return false;
  const bool scalar = p == 1 && n == 256;
  const bool long_rows = in > 6144;
  const int64_t above = g == 64          ? (scalar ? (long_rows ? 32 : 8) : (long_rows ? 48 : 16))
                        : g == 128 && scalar ? 32
                                             : 64;
  return batch > above;
}

extern "C" int higgs_internal_wide_plan(int64_t batch, int64_t out, int64_t in, int p, int n,
                                        int g, int64_t* splits) {
  if (!use_qgemm_wide(batch, in, p, n, g)) return -1;
  const WPlan plan = plan_wide(batch, out, in, g, pair_bits(p, n));
  *splits = plan.splits;
  return plan.shape;
}

int64_t qgemm_wide_workspace_bytes(int layers, int64_t batch, const int64_t* outs, int64_t in,
                                   int p, int n, int g) {
  return wide_layout(batch, outs, layers, layers, in, g, pair_bits(p, n)).total;
}

hipError_t launch_qgemm_wide(const void* x, int x_kind, int layers, const uint64_t* seeds,
                             int64_t batch, const uint8_t* const* codes,
                             const uint16_t* const* scales, const float* grid, int p, int n, int g,
                             const int64_t* outs, int64_t in, float* const* y, void* workspace,
                             hipStream_t stream) {
  bool same = true;
  for (int l = 1; l < layers; ++l) same = same && seeds[l] == seeds[0];
  const int nx = (x_kind == kQgemmRotated || same) ? 1 : layers;
  const int bits = pair_bits(p, n);
  const WLayout L = wide_layout(batch, outs, layers, nx, in, g, bits);
  char* ws = static_cast<char*>(workspace);
  _Float16* x16 = reinterpret_cast<_Float16*>(ws + L.x16);
  float* xe = reinterpret_cast<float*>(ws + L.xe);
  XSeeds xs{};
  xs.nl = nx;
  for (int l = 0; l < nx; ++l) xs.s[l] = seeds[l];
  hipError_t err;
  switch (x_kind) {
    case kQgemmRotated:
      err = launch_xprep_wide<float, false>(static_cast<const float*>(x), batch, in, g, xs, x16, xe,
                                            stream);
      break;
    case kQgemmRawF32:
      err = launch_xprep_wide<float, true>(static_cast<const float*>(x), batch, in, g, xs, x16, xe,
                                           stream);
      break;
    case kQgemmRawBF16:
      err = launch_xprep_wide<uint16_t, true>(static_cast<const uint16_t*>(x), batch, in, g, xs,
                                              x16, xe, stream);
      break;
    default:
      return hipErrorInvalidValue;
  }
  if (err != hipSuccess) return err;

  WPlan plan[kMaxGroup];
  float* part[kMaxGroup];
  for (int l = 0; l < layers; ++l) {
    plan[l] = plan_wide(batch, outs[l], in, g, bits);
    part[l] = plan[l].splits > 1 ? reinterpret_cast<float*>(ws + L.part[l]) : y[l];
  }
  int order[kMaxGroup];  // longest work items first
  for (int l = 0; l < layers; ++l) order[l] = l;
  std::stable_sort(order, order + layers,
                   [&](int a, int b) { return plan[a].kps > plan[b].kps; });
  // one launch per block shape that the layers use
  for (int shape = 0; shape < kShapes; ++shape) {
    QW a{};
    a.xe_stride = nx > 1 ? batch * (in / g) : 0;
    a.x16_stride = nx > 1 ? batch * in : 0;
    a.x16 = x16;
    a.xe = xe;
    a.grid = grid;
    a.batch = int(batch);
    a.pair_table = p == 1 ? 1 : 0;
    a.log2g = log2_exact(g);
    a.in = int(in);
    a.gpr = int(in / g);
    a.ctiles = int(ceil_div(batch, kShape[shape].cols));
    int64_t items = 0, turns = 0, run = 0;
    for (int i = 0; i < layers; ++i) {
      const int l = order[i];
      if (plan[l].shape != shape) continue;
      const int k = a.nl++;
      if (k == 0 || a.kps[k - 1] != int(plan[l].kps)) {
        turns += ceil_div(run, 8);
        run = 0;
        a.run0[k] = int(items);
      } else {
        a.run0[k] = a.run0[k - 1];
      }
      a.turn0[k] = int(turns);
      a.item0[k] = int(items);
      const int64_t n = ceil_div(outs[l], kShape[shape].rows) * plan[l].splits * a.ctiles;
      items += n;
      run += n;
      if (8 * turns + run >= (int64_t(1) << 31) - 8) return hipErrorInvalidValue;
      for (int j = 0; j <= k; ++j)
        if (a.run0[j] == a.run0[k]) a.run[j] = int(run);
      a.xcopy[k] = nx > 1 ? l : 0;
      a.kps[k] = int(plan[l].kps);
      a.splits[k] = int(plan[l].splits);
      a.out[k] = int(outs[l]);
      a.codes[k] = codes[l];
      a.scales[k] = scales[l];
      a.dst[k] = part[l];
    }
    if (a.nl == 0) continue;
    turns += ceil_div(run, 8);
    switch (bits) {
      case 6: err = launch_bits<6>(a, shape, unsigned(8 * turns), stream); break;
      case 8: err = launch_bits<8>(a, shape, unsigned(8 * turns), stream); break;
      case 10: err = launch_bits<10>(a, shape, unsigned(8 * turns), stream); break;
      case 16: err = launch_bits<16>(a, shape, unsigned(8 * turns), stream); break;
      default: return hipErrorInvalidValue;
    }
    if (err != hipSuccess) return err;
  }
  // the split layers' partial sums, all in one launch
  RG r{};
  r.nl = layers;
  for (int l = 0; l < layers; ++l) {
    r.part[l] = part[l];
    r.y[l] = y[l];
    r.n[l] = plan[l].splits > 1 ? batch * outs[l] : 0;
    r.splits[l] = int(plan[l].splits);
    r.off[l + 1] = r.off[l] + r.n[l];
  }
  if (r.off[layers] > 0) {
    const int64_t blocks = std::min<int64_t>((r.off[layers] + 255) / 256, 8192);
    hipLaunchKernelGGL(qgemm_reduce, dim3(unsigned(blocks)), dim3(256), 0, stream, r);
    return hipGetLastError();
  }
  return hipSuccess;
}

extern "C" void higgs_internal_wide_range(int in, int kps, int split, int groups, int q,
                                          int* first, int* stages, int* turns) {
  const WideRange r = wide_range(in, kps, split, groups, q);
  *first = r.first;
  *stages = r.stages;
  *turns = r.turns;
}

}  // namespace higgs
