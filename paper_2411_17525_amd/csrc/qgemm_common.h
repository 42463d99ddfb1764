// Pieces shared by the matrix-core products (qgemm.hip, qgemm_wide.hip): code
// formats and their lookup-table addressing, code loads, raw buffers, the sum of
// the K-splits.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"

namespace higgs {
namespace {

constexpr int kMaxGroup = 4;            // layers of one launch (they share the activations)

// Word 3 of a raw buffer resource on gfx9-family chips (32-bit data format).
constexpr int kRsrcWord3 = 0x00020000;
// Cache policy of the code loads: the default. A row's 128-byte line of
// codes is read in four pieces over four K-blocks (or super-blocks), so it
// must stay in L2 between them; with the non-temporal hint it was evicted
// early and a batch-64 product fetched 1.5-1.8x its code bytes.
constexpr int kAuxCodes = 0;
// Per-lane buffer offset beyond any buffer here (< 2^31 bytes): reads zero.
constexpr uint32_t kOffNone = 0x80000000u;

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f16x_acc __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x3 __attribute__((ext_vector_type(3)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// Code width: table copies (log2), log2 of a table entry's stride in bytes,
// code dwords per lane and K-block (16 codes), and whether codes are read as
// whole 128-byte lines and transposed through LDS (kCT, below).
// 8-bit: 32 copies in the low half of each 256-byte entry slot (64 KiB);
// the slots' high halves hold the code transposition rows. 6-bit: one copy
// per lane (16 KiB) and a separate transposition area. 10-bit: 16 copies
// (64 KiB). Scalar 8-bit codes: one copy per lane (64 KiB).
template <int BITS>
struct GFmt;
template <>
struct GFmt<8> {
  static constexpr int kRL = 5, kStride = 8, kWords = 4;
  static constexpr bool kCT = true;
};
template <>
struct GFmt<6> {
  static constexpr int kRL = 6, kStride = 8, kWords = 3;
  static constexpr bool kCT = true;
};
template <>
struct GFmt<10> {
  static constexpr int kRL = 4, kStride = 6, kWords = 5;
  static constexpr bool kCT = false;
};
// Scalar 8-bit codes (p = 1, n = 256): a pair of weights is two codes, each
// looked up on its own in a table of 256 single values (low half of the
// entry word, same addressing as the 8-bit pair codes).
template <>
struct GFmt<16> {
  static constexpr int kRL = 6, kStride = 8, kWords = 8;
  static constexpr bool kCT = false;
};

// Byte offset in the table of code c (0..15) of a lane's K-block for this
// lane's copy. 8-bit: one v_perm_b32 puts the code byte in byte 1 and the
// lane's copy offset (lane * 4 < 256) in byte 0, which is the address
// code * 256 + lane * 4 of a table with one copy per lane (entry stride 256
// bytes); otherwise the code's bit field, shifted to the entry stride,
// or'ed with copy * 4. lut_off_byte is the 8-bit form for byte b (0 ..
// 4 kWords - 1) of the lane's codes (scalar codes use it per weight).
template <int kWords>
__device__ inline uint32_t lut_off_byte(const uint32_t (&d)[kWords], int b, uint32_t copy_off) {
  const uint32_t sel = 0x0c0c0000u | (uint32_t(4 + (b & 3)) << 8);
  return __builtin_amdgcn_perm(d[b >> 2], copy_off, sel);
}

template <int BITS>
__device__ inline uint32_t lut_off(const uint32_t (&d)[GFmt<BITS>::kWords], int c,
                                   uint32_t copy_off) {
  if constexpr (BITS == 8) {
    return lut_off_byte<GFmt<8>::kWords>(d, c, copy_off);
  } else {
    constexpr int ST = GFmt<BITS>::kStride;
    const int bit = c * BITS, w = bit >> 5, o = bit & 31;
    uint32_t v;
    if (o + BITS <= 32)
      v = d[w] >> o;
    else
      v = __builtin_amdgcn_alignbit(d[w + 1], d[w], o);
    return ((v & ((1u << BITS) - 1u)) << ST) | copy_off;
  }
}

// One lane's codes of one K-block (kWords dwords at byte offset off).
template <int BITS>
__device__ inline void load_codes(__amdgpu_buffer_rsrc_t rs, uint32_t off,
                                  uint32_t (&d)[GFmt<BITS>::kWords]) {
  if constexpr (BITS == 8) {
    const i32x4 u = __builtin_amdgcn_raw_buffer_load_b128(rs, int(off), 0, kAuxCodes);
    d[0] = uint32_t(u.x); d[1] = uint32_t(u.y); d[2] = uint32_t(u.z); d[3] = uint32_t(u.w);
  } else if constexpr (BITS == 16) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const i32x4 u =
          __builtin_amdgcn_raw_buffer_load_b128(rs, int(off + 16u * q), 0, kAuxCodes);
      d[4 * q] = uint32_t(u.x); d[4 * q + 1] = uint32_t(u.y);
      d[4 * q + 2] = uint32_t(u.z); d[4 * q + 3] = uint32_t(u.w);
    }
  } else if constexpr (BITS == 6) {
    const i32x3 u = __builtin_amdgcn_raw_buffer_load_b96(rs, int(off), 0, kAuxCodes);
    d[0] = uint32_t(u.x); d[1] = uint32_t(u.y); d[2] = uint32_t(u.z);
  } else {
    const i32x4 u = __builtin_amdgcn_raw_buffer_load_b128(rs, int(off), 0, kAuxCodes);
    d[0] = uint32_t(u.x); d[1] = uint32_t(u.y); d[2] = uint32_t(u.z); d[3] = uint32_t(u.w);
    d[4] = uint32_t(__builtin_amdgcn_raw_buffer_load_b32(rs, int(off + 16u), 0, kAuxCodes));
  }
}

__device__ inline uint32_t pack_h2(float a, float b) {
  const _Float16 ha = static_cast<_Float16>(a), hb = static_cast<_Float16>(b);
  return uint32_t(__builtin_bit_cast(uint16_t, ha)) |
         (uint32_t(__builtin_bit_cast(uint16_t, hb)) << 16);
}

__device__ inline u32x4 as_u32x4(i32x4 v) {
  return u32x4{uint32_t(v.x), uint32_t(v.y), uint32_t(v.z), uint32_t(v.w)};
}

__device__ inline __amdgpu_buffer_rsrc_t rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, int(bytes), kRsrcWord3);
}

// Rotation seeds of the layers of one launch: layer l's activations go to
// copy l of the fp16 buffer and to xe + l * ngroups (one copy per layer when
// the layers rotate with their own seeds; nl = 1 when they share the copy).
struct XSeeds {
  uint64_t s[kMaxGroup];
  int nl;
};

// The layers' partial products of one launch: layer l's [splits[l]][n[l]]
// at part[l], its output (n[l] floats) at y[l]; off[l] = n[0] + ... +
// n[l - 1]. A layer without a K-split has n[l] = 0 (its product wrote y), so
// index i belongs to the last layer l with off[l] <= i.
struct RG {
  const float* part[kMaxGroup];
  float* y[kMaxGroup];
  int64_t n[kMaxGroup];
  int64_t off[kMaxGroup + 1];
  int splits[kMaxGroup];
  int nl;
};

// y = sum over splits of the partial products, in split order.
__global__ __launch_bounds__(256) void qgemm_reduce(const RG r) {
  // every argument in one round trip; the layer of an index is then picked
  // by selects (an indexed read would be a second round trip)
  const float* part_l[kMaxGroup];
  float* y_l[kMaxGroup];
  int64_t n_l[kMaxGroup], off_l[kMaxGroup + 1];
  int splits_l[kMaxGroup];
#pragma unroll
  for (int l = 0; l < kMaxGroup; ++l) {
    part_l[l] = r.part[l];
    y_l[l] = r.y[l];
    n_l[l] = r.n[l];
    off_l[l] = r.off[l];
    splits_l[l] = r.splits[l];
  }
  off_l[kMaxGroup] = r.off[kMaxGroup];
  const int nl = r.nl;
  static_assert(kMaxGroup == 4, "the read below names four layers");
  HIGGS_READ_NOW("s"(part_l[0]), "s"(part_l[1]), "s"(part_l[2]), "s"(part_l[3]), "s"(y_l[0]),
                 "s"(y_l[1]), "s"(y_l[2]), "s"(y_l[3]), "s"(n_l[0]), "s"(n_l[1]), "s"(n_l[2]),
                 "s"(n_l[3]), "s"(off_l[1]), "s"(off_l[2]), "s"(off_l[3]), "s"(off_l[4]),
                 "s"(splits_l[0]), "s"(splits_l[1]), "s"(splits_l[2]), "s"(splits_l[3]),
                 "s"(nl), "s"(gridDim.x));
  int64_t total = off_l[1];
#pragma unroll
  for (int l = 2; l <= kMaxGroup; ++l)
    if (l == nl) total = off_l[l];
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < total;
       i += int64_t(gridDim.x) * 256) {
    int L = 0;
#pragma unroll
    for (int l = 1; l < kMaxGroup; ++l)
      if (l < nl && i >= off_l[l]) L = l;
    const float* part = part_l[0];
    float* y = y_l[0];
    int64_t n = n_l[0], j = i;
    int splits = splits_l[0];
#pragma unroll
    for (int l = 1; l < kMaxGroup; ++l)
      if (L == l) {
        part = part_l[l];
        y = y_l[l];
        n = n_l[l];
        j = i - off_l[l];
        splits = splits_l[l];
      }
    // loads eight splits at a time (one memory round trip for up to eight),
    // adds in split order starting from split 0's value
    float s = 0.f;
    for (int k = 0; k < splits; k += 8) {
      float v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = part[int64_t(min(k + q, splits - 1)) * n + j];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (k + q < splits) s = k + q == 0 ? v[q] : s + v[q];
    }
    y[j] = s;
  }
}

}  // namespace
}  // namespace higgs
