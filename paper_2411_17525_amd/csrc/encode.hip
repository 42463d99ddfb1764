// HIGGS encoder (Alg. 1, RHT-VQ, with the grid of Alg. 2) on the GPU.
//
// Per group of g consecutive weights of one row (a wavefront takes 1024 weights
// at a time, 1024 / g groups of up to 1024):
//   s = ||w||_2                      (fp64 sum of squares, fixed reduction tree)
//   w_dag = H (sigma * (w / s))      (fp64, in-register / cross-lane butterflies)
//   code_j = argmin_k ||w_dag[jp:(j+1)p] - G_k||^2, lowest k on ties
//   scale = fp16(s / sqrt(g))        (one rounding from fp64)
// The search compares c_k = |G_k|^2 / 2 - <v, G_k>, which orders the grid
// points exactly as the squared distance does, in fp64. To take the running
// minimum and its index in one v_min_f64, each candidate's value is shifted
// by a power of two S that makes it positive and its 10 lowest mantissa bits
// are replaced by k: positive doubles order as their bit patterns, so the
// minimum is the smallest value, ties (and values within 1024 ulps of S,
// S 2^-42) going to the lowest k. |v| <= sqrt(g) for a p-vector of a rotated
// group (its squared norm sums to g), so |c_k| <= R^2 / 2 + sqrt(g) R with R
// the largest grid-point norm; each block takes S = the least power of two
// >= max(1024, 2 (R^2 / 2 + sqrt(g) R)) from the grid it loads. Every grid of
// unit-variance points gets S = 1024, where the order differs from the plain
// fp64 distance only at squared-distance gaps below ~5e-10; the band is
// S 2^-41 in general, below 1e-6 for grids whose points have norms <= 1024.
// Candidates: with a search index built from the same grid, a p-vector is
// compared with the grid points of its bucket's list only (exact pruning,
// below), which holds every point whose search value can be the least one
// for a vector in that bucket; vectors outside the bucketed square, and every
// vector without a matching index, scan all n points. The chosen code is the
// one a full scan gives.
// Codes are packed LSB-first into the row's bit stream through LDS.

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.h"
#include "wave_fwht.h"

namespace higgs {
namespace {

constexpr int kWaves = 4;
constexpr int kMaxN = 1024;
constexpr int kMaxG = 4096;
constexpr double kMinShift = 1024.0;   // least shift of the search values
constexpr uint32_t kIndexMask = 1023;  // low mantissa bits that carry the index (n <= 1024)

// min(best, c with its 10 lowest mantissa bits replaced by k). c and best
// are positive and finite, so no NaN handling is needed: one bit-field insert
// on the low word and one v_min_f64 (the compiler's fmin would first quieten
// both operands).
__device__ inline double min_indexed(double best, double c, uint32_t k, uint32_t index_mask) {
  const uint64_t u = __builtin_bit_cast(uint64_t, c);
  uint32_t lo;
  // lo = (k & index_mask) | (low word of c & ~index_mask); index_mask in a VGPR
  __asm__("v_bfi_b32 %0, %1, %2, %3" : "=v"(lo) : "v"(index_mask), "s"(k), "v"(uint32_t(u)));
  const double ck = __builtin_bit_cast(double, (u & 0xffffffff00000000ull) | uint64_t(lo));
  double r;
  __asm__("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(best), "v"(ck));
  return r;
}

// fp64 -> IEEE binary16 bits, round to nearest even, for finite x >= 0.
__device__ inline uint16_t f64_to_f16_rne(double x) {
  if (!(x > 0.0)) return 0;
  if (x >= 65520.0) return 0x7C00;                  // rounds to +infinity
  const int e = ilogb(x);                           // x in [2^e, 2^(e+1))
  const int qe = e - 10 > -24 ? e - 10 : -24;       // fp16 spacing in that binade
  const double r = ldexp(rint(ldexp(x, -qe)), qe);  // exact fp16 value
  const _Float16 h = static_cast<_Float16>(static_cast<float>(r));  // exact conversions
  return __builtin_bit_cast(uint16_t, h);
}

template <typename InT>
__device__ inline double to_f64(InT v);
template <>
__device__ inline double to_f64<float>(float v) { return double(v); }
template <>
__device__ inline double to_f64<uint16_t>(uint16_t v) {
  return double(__uint_as_float(uint32_t(v) << 16));
}

template <int E, typename InT>
__device__ inline void load_group(const InT* __restrict__ src, double (&v)[E]) {
  constexpr int kBytes = E * int(sizeof(InT));
  if constexpr (kBytes % 16 == 0) {
    constexpr int kPer = 16 / int(sizeof(InT));
#pragma unroll
    for (int q = 0; q < kBytes / 16; ++q) {
      const u32x4 u = load_stream16(reinterpret_cast<const char*>(src) + 16 * q);
      const InT* e = reinterpret_cast<const InT*>(&u);
#pragma unroll
      for (int i = 0; i < kPer; ++i) v[q * kPer + i] = to_f64<InT>(e[i]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = to_f64<InT>(src[i]);
  }
}

// The same in two parts, so that a group's loads can be issued while the one
// before it is worked on: the values as they lie in memory, then in fp64.
template <int E, typename InT>
struct RawGroup {
  static constexpr int kBytes = E * int(sizeof(InT));
  static constexpr bool kVec = kBytes % 16 == 0;
  u32x4 u[kVec ? kBytes / 16 : 1];
  InT e[kVec ? 1 : E];
  __device__ inline void load(const InT* __restrict__ src) {
    if constexpr (kVec) {
#pragma unroll
      for (int q = 0; q < kBytes / 16; ++q)
        u[q] = load_stream16(reinterpret_cast<const char*>(src) + 16 * q);
    } else {
#pragma unroll
      for (int i = 0; i < E; ++i) e[i] = src[i];
    }
  }
  // flips signs (masks below)
  __device__ inline void flip(const uint32_t (&mask)[kVec ? kBytes / 4 : E]) {
    if constexpr (kVec) {
#pragma unroll
      for (int q = 0; q < kBytes / 16; ++q)
        u[q] ^= u32x4{mask[4 * q], mask[4 * q + 1], mask[4 * q + 2], mask[4 * q + 3]};
    } else {
#pragma unroll
      for (int i = 0; i < E; ++i) {
        if constexpr (sizeof(InT) == 4)
          e[i] = __uint_as_float(__float_as_uint(e[i]) ^ mask[i]);
        else
          e[i] = InT(e[i] ^ InT(mask[i]));
      }
    }
  }
  static constexpr int kMasks = kVec ? kBytes / 4 : E;
  // flip's masks for sign bits neg of the lane's elements
  __device__ static inline void masks(uint64_t neg, uint32_t (&mask)[kMasks]) {
#pragma unroll
    for (int i = 0; i < kMasks; ++i) {
      if constexpr (sizeof(InT) == 4)
        mask[i] = uint32_t(neg >> i) << 31;
      else if constexpr (kVec)
        mask[i] = (uint32_t(neg >> (2 * i)) & 1u) << 15 | uint32_t(neg >> (2 * i + 1)) << 31;
      else
        mask[i] = (uint32_t(neg >> i) & 1u) << 15;
    }
  }
  __device__ inline void expand(double (&v)[E]) const {
    if constexpr (kVec) {
#pragma unroll
      for (int q = 0; q < kBytes / 16; ++q) {
        const uint32_t w[4] = {u[q].x, u[q].y, u[q].z, u[q].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if constexpr (sizeof(InT) == 4) {
            v[4 * q + k] = double(__uint_as_float(w[k]));
          } else {
            v[8 * q + 2 * k] = double(__uint_as_float(w[k] << 16));
            v[8 * q + 2 * k + 1] = double(__uint_as_float(w[k] & 0xffff0000u));
          }
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = to_f64<InT>(e[i]);
    }
  }
};

// ---------------------------------------------------------------------------
// Search index: exact pruning of the nearest-point search. The square
// [-kBR, kBR)^P is cut into kNB^P buckets. Point k may be left out of bucket
// B's list when some point j is nearer than k to every point of B, by a
// margin m in squared distance: dmin(k, B)^2 > dmax(j, B)^2 + m, with dmin /
// dmax the least and the largest distance from the point to the (slightly
// widened) box of B. Since c_k - c_j = (|v - G_k|^2 - |v - G_j|^2) / 2, such
// a k has a search value above j's by more than m / 2 for every v in B; m
// (2^-30 S, S the search shift of the largest group size, which bounds the
// shift of every group size) is far above the 2^-42 S by which the index
// bits move a value and the rounding of the values, so k is never the least
// one. A list is never empty: it holds the point that sets the bound.
//
// The index is built once per grid (one wavefront per bucket, then one block
// that lays the lists out back to back) and read by every quantize block into
// LDS. It carries a hash of the grid's values, the margin and its geometry;
// a block that loads a grid whose hash differs, or an index that is missing
// or does not fit, scans all n points for every vector, so an index can only
// change the speed of a call, never its codes.
// ---------------------------------------------------------------------------
constexpr double kBR = 4.0;      // half side of the bucketed square
constexpr double kBEps = 1e-9;   // widening of a bucket's box (bucket-index rounding)
constexpr uint32_t kIndexMagic = 0x49534748u;
constexpr int kSlotCap = 64;     // entries per bucket while the index is built
// Buckets per axis: 512 for p = 1; for p = 2, 64 (128 for the 1024-point
// grid, whose lists would average about 9 points at 64: 3 at 128).
__host__ __device__ constexpr int index_nb(int p, int n) {
  return p == 1 ? 512 : (n >= 256 ? 128 : 64);
}
__host__ __device__ constexpr int index_cells(int p, int n) {
  return p == 1 ? index_nb(p, n) : index_nb(p, n) * index_nb(p, n);
}
template <int P, int N>
struct Buckets {
  static constexpr int kNB = index_nb(P, N), kCells = index_cells(P, N);
};

__host__ __device__ constexpr int64_t align16(int64_t b) { return (b + 15) / 16 * 16; }
// list entries a quantize block holds in LDS
__host__ __device__ constexpr int index_list_cap(int p, int n) {
  return p == 1 ? 2048 : (n <= 64 ? 8192 : 32768);
}

struct IndexHeader {
  uint32_t magic, p, n, nb;
  uint32_t total, usable, reserved0, reserved1;
  uint64_t hash;
  double margin, half_side;
  uint64_t reserved;
};
static_assert(sizeof(IndexHeader) == 64, "index header");

// header | u16 offsets [cells + 1] | u16 lists [cap] | build scratch: u16
// counts [cells], u16 slots [cells][kSlotCap]; regions 16-byte aligned
struct IndexLayout {
  int64_t offsets, list, counts, slots, bytes;
};
__host__ __device__ constexpr IndexLayout index_layout(int p, int n) {
  const int64_t cells = index_cells(p, n);
  const int64_t offsets = 64;
  const int64_t list = offsets + align16((cells + 1) * 2);
  const int64_t counts = list + align16(int64_t(index_list_cap(p, n)) * 2);
  const int64_t slots = counts + align16(cells * 2);
  return IndexLayout{offsets, list, counts, slots, slots + cells * kSlotCap * 2};
}

// the search-value shift for groups of g weights: a power of two at least
// twice the largest |c_k| (see the file's header)
__device__ inline double search_shift(double r2, int g) {
  const double bound = 2.0 * (0.5 * r2 + sqrt(double(g)) * sqrt(r2));
  return bound <= kMinShift ? kMinShift : exp2(ceil(log2(bound)));
}

// hash of grid point k (its index and the bits of its coordinates); the
// grid's hash is the sum over its points (mod 2^64)
template <int P>
__device__ inline uint64_t point_hash(const float* c, int k) {
  uint64_t h = splitmix64_at(0x48474753ull, uint64_t(k));
#pragma unroll
  for (int t = 0; t < P; ++t) h = splitmix64_at(h, __float_as_uint(c[t]));
  return h;
}

// dmin^2 and dmax^2 from point g to the box [lo, lo + w]^P (widened by kBEps)
template <int P>
__device__ inline void box_d2(const double* g, const double (&lo)[P], double w, double& dmin2,
                              double& dmax2) {
  dmin2 = 0.0;
  dmax2 = 0.0;
#pragma unroll
  for (int t = 0; t < P; ++t) {
    const double a = lo[t] - kBEps - g[t], b = g[t] - (lo[t] + w + kBEps);
    const double dn = fmax(0.0, fmax(a, b));
    const double dx = fmax(fabs(a), fabs(b));
    dmin2 = fma(dn, dn, dmin2);
    dmax2 = fma(dx, dx, dmax2);
  }
}

// Vectors with every |v| below this walk their bucket's list. Less than kBR by
// the boxes' widening: the largest double below kBR would round up to the bucket
// past the last one.
constexpr double kBIn = kBR - kBEps;

// Bucket index along one axis for |v| < kBIn: floor((v + kBR) nb / (2 kBR)) as
// the nearest integer to that value less 1/2, read from the low mantissa bits
// after adding 3 2^51 (no change of binade around it). On a bucket's edge it
// may name either neighbour, and its roundings are below 1e-12: both are
// covered by the widening of the boxes.
__device__ inline int bucket_axis(double v, int nb) {
  const double f = fma(v, double(nb) / (2.0 * kBR), 0.5 * double(nb) - 0.5) + 0x1.8p52;
  return int(uint32_t(__builtin_bit_cast(uint64_t, f)));
}

// In place: counts a[0 .. n) -> exclusive offsets, a[n] = total (n + 1
// entries; block-wide, every thread of the block calls it). Returns the
// total (every thread). s_tmp: one entry per wave.
__device__ inline int block_offsets(uint32_t* a, int n, int tid, int nthreads, uint32_t* s_tmp) {
  const int per = (n + nthreads - 1) / nthreads;
  const int b0 = min(n, tid * per), b1 = min(n, b0 + per);
  uint32_t local = 0;
  for (int i = b0; i < b1; ++i) local += a[i];
  // inclusive scan over the wave
  const int lane = tid & 63, wave = tid >> 6;
  uint32_t inc = local;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = uint32_t(__shfl_up(int(inc), d));
    if (lane >= d) inc += o;
  }
  if (lane == 63) s_tmp[wave] = inc;
  __syncthreads();
  uint32_t base = 0, total = 0;
  for (int w = 0; w < nthreads / 64; ++w) {
    if (w < wave) base += s_tmp[w];
    total += s_tmp[w];
  }
  uint32_t run = base + inc - local;
  for (int i = b0; i < b1; ++i) {
    const uint32_t c = a[i];
    a[i] = run;
    run += c;
  }
  if (tid == 0) a[n] = total;
  __syncthreads();
  return int(total);
}

// One wavefront per bucket: the bucket's list into its slot (at most
// kSlotCap entries kept, the full count written).
template <int P, int N>
__global__ __launch_bounds__(256) void index_slots_kernel(const float* __restrict__ grid, int n,
                                                          uint8_t* __restrict__ index) {
  using B = Buckets<P, N>;
  constexpr double kW = 2.0 * kBR / B::kNB;
  const IndexLayout L = index_layout(P, n);
  const int lane = int(threadIdx.x) & 63;
  const int b = int(blockIdx.x) * 4 + (int(threadIdx.x) >> 6);
  if (b >= B::kCells) return;  // whole waves
  double lo[P];
  lo[0] = -kBR + kW * (b % B::kNB);
  if constexpr (P == 2) lo[1] = -kBR + kW * (b / B::kNB);
  // the margin, from the largest squared norm; the bound u = min_j dmax^2
  double r2 = 0.0, u = INFINITY;
  for (int k = lane; k < n; k += 64) {
    double gk[P], h = 0.0;
#pragma unroll
    for (int t = 0; t < P; ++t) {
      gk[t] = double(grid[k * P + t]);
      h += gk[t] * gk[t];
    }
    r2 = fmax(r2, h);
    double dn, dx;
    box_d2<P>(gk, lo, kW, dn, dx);
    u = fmin(u, dx);
  }
  r2 = wave_max(r2, lane);
  u = -wave_max(-u, lane);
  const double m = ldexp(search_shift(r2, kMaxG), -30);
  uint16_t* slot = reinterpret_cast<uint16_t*>(index + L.slots) + int64_t(b) * kSlotCap;
  uint32_t cnt = 0;
  for (int k0 = 0; k0 < n; k0 += 64) {
    const int k = k0 + lane;
    bool take = false;
    if (k < n) {
      double gk[P];
#pragma unroll
      for (int t = 0; t < P; ++t) gk[t] = double(grid[k * P + t]);
      double dn, dx;
      box_d2<P>(gk, lo, kW, dn, dx);
      take = dn <= u + m;
    }
    const uint64_t bal = __ballot(take);
    if (take) {
      const uint32_t at = cnt + uint32_t(__popcll(bal & ((uint64_t(1) << lane) - 1)));
      if (at < uint32_t(kSlotCap)) slot[at] = uint16_t(k);
    }
    cnt += uint32_t(__popcll(bal));
  }
  if (lane == 0)
    reinterpret_cast<uint16_t*>(index + L.counts)[b] = uint16_t(cnt < 65535u ? cnt : 65535u);
}

// One block of 1024 threads: offsets, the lists back to back, the header.
template <int P, int N>
__global__ __launch_bounds__(1024) void index_finish_kernel(const float* __restrict__ grid, int n,
                                                            uint8_t* __restrict__ index) {
  using B = Buckets<P, N>;
  constexpr int kThreads = 1024;
  const IndexLayout L = index_layout(P, n);
  __shared__ uint32_t s_off[B::kCells + 1];
  __shared__ uint32_t s_tmp[kThreads / 64];
  __shared__ uint64_t s_hash[kThreads / 64];
  __shared__ double s_r2[kThreads / 64];
  __shared__ int s_over;
  const int tid = int(threadIdx.x), lane = tid & 63, wave = tid >> 6;
  const uint16_t* counts = reinterpret_cast<const uint16_t*>(index + L.counts);
  const uint16_t* slots = reinterpret_cast<const uint16_t*>(index + L.slots);
  if (tid == 0) s_over = 0;
  __syncthreads();
  for (int b = tid; b < B::kCells; b += kThreads) {
    const uint32_t c = counts[b];
    if (c > uint32_t(kSlotCap)) s_over = 1;
    s_off[b] = c;
  }
  __syncthreads();
  const int total = block_offsets(s_off, B::kCells, tid, kThreads, s_tmp);
  const bool usable = s_over == 0 && total <= index_list_cap(P, n);
  uint16_t* offs = reinterpret_cast<uint16_t*>(index + L.offsets);
  uint16_t* list = reinterpret_cast<uint16_t*>(index + L.list);
  for (int b = tid; b <= B::kCells; b += kThreads) offs[b] = usable ? uint16_t(s_off[b]) : 0;
  if (usable) {
    for (int b = tid; b < B::kCells; b += kThreads) {
      const uint32_t o = s_off[b], c = s_off[b + 1] - o;
      for (uint32_t e = 0; e < c; ++e) list[o + e] = slots[int64_t(b) * kSlotCap + e];
    }
  }
  uint64_t h = 0;
  double r2 = 0.0;
  for (int k = tid; k < n; k += kThreads) {
    float c[P];
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < P; ++t) {
      c[t] = grid[k * P + t];
      s += double(c[t]) * double(c[t]);
    }
    h += point_hash<P>(c, k);
    r2 = fmax(r2, s);
  }
  h = wave_sum(h, lane);
  r2 = wave_max(r2, lane);
  if (lane == 0) {
    s_hash[wave] = h;
    s_r2[wave] = r2;
  }
  __syncthreads();
  if (tid == 0) {
    uint64_t hs = 0;
    double rr = 0.0;
    for (int w = 0; w < kThreads / 64; ++w) {
      hs += s_hash[w];
      rr = fmax(rr, s_r2[w]);
    }
    IndexHeader hd{};
    hd.magic = kIndexMagic;
    hd.p = P;
    hd.n = uint32_t(n);
    hd.nb = B::kNB;
    hd.total = usable ? uint32_t(total) : 0u;
    hd.usable = usable ? 1u : 0u;
    hd.hash = hs;
    hd.margin = ldexp(search_shift(rr, kMaxG), -30);
    hd.half_side = kBR;
    *reinterpret_cast<IndexHeader*>(index) = hd;
  }
}

// min(a, b) of values that are not NaN (fmin would first quieten both).
__device__ inline double min_f64(double a, double b) {
  double r;
  __asm__("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Minimum over the 64 lanes of the wave, in every lane (no NaNs).
__device__ inline double wave_min(double v, int lane) {
  v = min_f64(v, lane_xor<32>(v, lane));
  v = min_f64(v, lane_xor<16>(v, lane));
  v = min_f64(v, lane_xor<8>(v, lane));
  v = min_f64(v, lane_xor<4>(v, lane));
  v = min_f64(v, lane_xor<2>(v, lane));
  v = min_f64(v, lane_xor<1>(v, lane));
  return v;
}

__device__ inline double readlane_f64(double v, int l) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u)), l));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u >> 32)), l));
  return __builtin_bit_cast(double, uint64_t(lo) | (uint64_t(hi) << 32));
}

// grid point in LDS: its coordinates as read (fp32, exact in fp64), one
// 8-byte read per candidate; the search constant is formed in registers
struct __align__(8) GridPt {
  float x[2];
};

// |G_k|^2 / 2 + S in fp64: the squares are exact, then one rounding for
// their sum (p = 2) and one for adding S (half the sum is exact)
template <int P>
__device__ inline double search_const(const GridPt& q, double shift) {
  double h = double(q.x[0]) * double(q.x[0]);
  if constexpr (P == 2) h = fma(double(q.x[1]), double(q.x[1]), h);
  return fma(0.5, h, shift);
}

// Sum of v over the lane's aligned run of L lanes, in every lane of it (for
// L = 64 in wave_sum's order).
template <int L>
__device__ inline double lanes_sum(double v, int lane) {
  if constexpr (L > 32) v += lane_xor<32>(v, lane);
  if constexpr (L > 16) v += lane_xor<16>(v, lane);
  if constexpr (L > 8) v += lane_xor<8>(v, lane);
  if constexpr (L > 4) v += lane_xor<4>(v, lane);
  if constexpr (L > 2) v += lane_xor<2>(v, lane);
  if constexpr (L > 1) v += lane_xor<1>(v, lane);
  return v;
}

__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sign bits of the group's elements (bit j of word q: element 64 q + j is
// negated), computed by all the waves of the block. Ends with a barrier.
template <int E, int kNW>
__device__ inline void block_signs(uint64_t seed, uint64_t (&s_neg)[E], int wave, int lane) {
  for (int q = wave; q < E; q += kNW) {
    const uint64_t bits = __ballot(rht_sign_negative(seed, uint32_t(64 * q + lane)));
    if (lane == 0) s_neg[q] = bits;
  }
  __syncthreads();
}

// Copies `bytes` (a multiple of 16) of device memory to LDS by the kQW waves of
// a block, with no registers between; complete after the waves' own wait for
// vector memory and a block barrier.
template <int kQW>
__device__ inline void copy_to_lds(const uint8_t* src, void* dst, int bytes, int wave, int lane) {
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(src), 0, bytes, 0x00020000);
  for (int o = wave * 1024; o < bytes; o += kQW * 1024)
    if (o + lane * 16 < bytes)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (__attribute__((address_space(3))) void*)(static_cast<char*>(dst) + o), 16,
          o + lane * 16, 0, 0, 0);
}

// Bound by the vector ALU (about 1200 instructions per 1024 weights and lane,
// busy 77% of the time at 14336 x 4096, 256 points, bf16: 155 us, 250 before):
// the fp64 rotation is a third, the walk of the lists (12 instructions per
// candidate, four candidates deep) another. The prologue's index arrives in one
// memory round trip (1024 x 1024: 41 us before, 15 now).
// G: group size (64 .. 1024); P: grid dimension; BITS: packed code width; kQW:
// waves per block. A wave takes 1024 weights at a time, 1024 / G groups of them
// (16 weights per lane whatever the group size: with G / 64 per lane, small
// groups left a lane one or two vectors, and every read of their search waited
// on its own; 4096 x 4096 fp32, 1024 points, G = 256: 97 us
// against 87; 256-point scalar grid, G = 128: 88 against 45). The waves of a
// block share the grid and the index in LDS and then take their weights
// independently (no block barrier after the prologue). Without an index and
// with few weights (`shared`: the block's waves would leave half the chip idle)
// all the waves of a block take the same 1024 weights, each scans its part of
// the points, and the first one writes the least: 16 x 4096 bf16 with 256 scalar
// points, g = 64: 62 us -> 13, 1024 points, g = 128: 246 -> 28.
template <int G, int P, int BITS, int kQW, typename InT>
__global__ __launch_bounds__(64 * kQW) void quantize_kernel(
    const InT* __restrict__ w, int64_t groups, uint64_t seed, const float* __restrict__ grid, int n,
    const uint8_t* __restrict__ index, bool shared, uint8_t* __restrict__ codes,
    uint16_t* __restrict__ scales) {
  constexpr int E = 16;           // weights per lane
  constexpr int kSeg = 64 * E;    // per wave and turn
  constexpr int kSegGroups = kSeg / G;
  constexpr int kGroupLanes = G / E;
  constexpr int kVecPerLane = E / P;
  constexpr int kSegCodes = kSeg / P;
  constexpr int kWordsPerGroup = G / P * BITS / 32;
  constexpr int kN = 1 << BITS;  // grid points of the format (the host passes n = 2^BITS)
  static_assert(kN <= kMaxN, "grid size");
  using BK = Buckets<P, kN>;
  constexpr int kCap = index_list_cap(P, kN);
  constexpr IndexLayout kL = index_layout(P, kN);
  using CodeT = typename std::conditional<(BITS <= 8), uint8_t, uint16_t>::type;

  // whether the waves of a block can share their weights (a scan of few points
  // is short)
  constexpr bool kShare = kN > 16;
  // their values take the place of the lists, where those are large
  constexpr bool kInList = kCap * 2 >= kSegCodes * 8;

  // the rotation's scratch, which then takes the codes
  static_assert(kFwhtRows * 4 >= int(kSegCodes * sizeof(CodeT)), "codes fit the scratch");
  __shared__ GridPt s_grid[kN];
  __shared__ __align__(16) uint32_t s_scratch[kQW][kFwhtRows];
  __shared__ uint64_t s_neg[G / 64];
  __shared__ __align__(16) uint16_t s_off[align16((BK::kCells + 1) * 2) / 2];
  __shared__ __align__(16) uint16_t s_list[kCap];
  __shared__ unsigned long long s_values[kShare && !kInList ? kSegCodes : 1];
  __shared__ double s_r2[kQW];
  __shared__ uint64_t s_hash[kQW];

  const int tid = int(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // The index's offsets and lists straight into LDS, and its header, all
  // requested before anything else is done (an index holds these regions
  // whatever its header says): read after the header's checks, field by field
  // and through registers, they took a dozen memory round trips per block.
  u32x4 hdr[4] = {};
  if (index != nullptr) {
    copy_to_lds<kQW>(index + kL.offsets, s_off, int(sizeof(s_off)), wave, lane);
    copy_to_lds<kQW>(index + kL.list, s_list, int(sizeof(s_list)), wave, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) hdr[q] = reinterpret_cast<const u32x4*>(index)[q];
  }

  // the grid, its largest squared norm and (with an index) its hash
  double r2 = 0.0;
  uint64_t hsh = 0;
  for (int k = tid; k < n; k += 64 * kQW) {
    float c[P];
    double h = 0.0;
#pragma unroll
    for (int t = 0; t < P; ++t) {
      c[t] = grid[k * P + t];
      h += double(c[t]) * double(c[t]);
    }
    GridPt q;
    q.x[0] = c[0];
    q.x[1] = P == 2 ? c[P - 1] : 0.0f;
    s_grid[k] = q;
    r2 = fmax(r2, h);
    if (index != nullptr) hsh += point_hash<P>(c, k);
  }
  r2 = wave_max(r2, lane);
  hsh = wave_sum(hsh, lane);
  if (lane == 0) {
    s_r2[wave] = r2;
    s_hash[wave] = hsh;
  }
  __syncthreads();
  hsh = 0;
  for (int i = 0; i < kQW; ++i) {
    r2 = fmax(r2, s_r2[i]);
    hsh += s_hash[i];
  }
  const double shift = search_shift(r2, G);

  // the index counts when it was built from this grid and fits
  static_assert(sizeof(hdr) == sizeof(IndexHeader), "header");
  const IndexHeader hd = __builtin_bit_cast(IndexHeader, hdr);
  const bool pruned =
      index != nullptr &&
      ((hd.magic == kIndexMagic) & (hd.p == uint32_t(P)) & (hd.n == uint32_t(n)) &
       (hd.nb == uint32_t(BK::kNB)) & (hd.usable == 1u) & (hd.total <= uint32_t(kCap)) &
       (hd.hash == hsh) & (hd.half_side == kBR) & (hd.margin >= ldexp(shift, -30)));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the copies into LDS

  block_signs<G / 64, kQW>(seed, s_neg, wave, lane);  // (its barrier also covers the index)
  uint32_t flips[RawGroup<E, InT>::kMasks];
  const int in_group = lane * E % G;  // the lane's first weight inside its group
  RawGroup<E, InT>::masks(s_neg[in_group / 64] >> (in_group % 64), flips);

  const double inv_sqrt_g = 1.0 / sqrt(double(G));
  const uint32_t index_mask = kIndexMask;
  CodeT* const s_codes = reinterpret_cast<CodeT*>(s_scratch[wave]);
  // place, in the wave's 1024 weights, of the code of the lane's first vector
  // after the rotation (and, for P = 2, the exchange below)
  const int code0 = P == 2 ? (fwht_rows_lane<G>(lane & ~1) >> 1) | (lane & 1) << 3
                           : fwht_rows_lane<G>(lane);

  // groups, their scales and their codes all lie back to back; the next turn's
  // weights are requested one turn ahead. Past the last group a lane has zeros.
  const int64_t segs = (groups + kSegGroups - 1) / kSegGroups;
  const int64_t step = shared ? int64_t(gridDim.x) : int64_t(gridDim.x) * kQW;
  int64_t seg = shared ? int64_t(blockIdx.x) : int64_t(blockIdx.x) * kQW + wave;
  RawGroup<E, InT> raw = {};
  auto request = [&](int64_t sg) {
    if (kSegGroups == 1 || sg * kSegGroups + lane / kGroupLanes < groups)
      raw.load(w + sg * kSeg + lane * E);
    else
      raw = RawGroup<E, InT>{};
  };
  if (seg < segs) request(seg);
  for (; seg < segs; seg += step) {
    double v[E];
    raw.flip(flips);  // sigma
    raw.expand(v);
    if (seg + step < segs) request(seg + step);

    double ss = 0.0;
#pragma unroll
    for (int i = 0; i < E; ++i) ss += v[i] * v[i];
    ss = lanes_sum<kGroupLanes>(ss, lane);  // over the group's lanes
    const double s = sqrt(ss);

    // w / s as w * (1 / s): within an ulp of the quotient
    const double inv_s = s > 0.0 ? 1.0 / s : 0.0;
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] *= inv_s;
    fwht_rows<G>(v, s_scratch[wave], lane);
    if constexpr (P == 2) {
      // a vector's two coordinates are in lanes l and l ^ 1: exchange lane bit
      // 0 with register bit 0, so that lane l has the vector of registers 2 q
      // (even l) or 2 q + 1 (odd l) in v[2 q], v[2 q + 1]
      const bool odd = lane & 1;
#pragma unroll
      for (int q = 0; q < E / 2; ++q) {
        const double x = v[2 * q], y = v[2 * q + 1];
        const double got = lane_xor<1>(odd ? x : y, lane);
        v[2 * q] = odd ? got : x;
        v[2 * q + 1] = odd ? y : got;
      }
    }

    // search value of point k for vector j, folded into best[j]
    double best[kVecPerLane];
#pragma unroll
    for (int j = 0; j < kVecPerLane; ++j) best[j] = INFINITY;
    auto fold = [&](int j, int k, const GridPt& q) {
      double c = fma(-v[j * P], double(q.x[0]), search_const<P>(q, shift));
      if constexpr (P == 2) c = fma(-v[j * P + 1], double(q.x[1]), c);
      best[j] = min_indexed(best[j], c, uint32_t(k), index_mask);
    };
    // vectors that scan every point (one bit per vector of the lane)
    uint64_t full = (uint64_t(1) << kVecPerLane) - 1;
    if (pruned) {
      // the vectors' lists, walked side by side (a list that ends repeats
      // its last entry, which leaves the minimum unchanged)
      int at[kVecPerLane], last[kVecPerLane];
      int steps = 0;
#pragma unroll
      for (int j = 0; j < kVecPerLane; ++j) {
        bool in_box = fabs(v[j * P]) < kBIn;  // (false for NaN)
        int b = bucket_axis(v[j * P], BK::kNB);
        if constexpr (P == 2) {
          in_box = in_box && fabs(v[j * P + 1]) < kBIn;
          b += bucket_axis(v[j * P + 1], BK::kNB) * BK::kNB;
        }
        b = in_box ? b : 0;  // (its list is walked all the same)
        const int o = s_off[b], e = s_off[b + 1];
        at[j] = o;
        last[j] = e - o - 1;
        if (in_box) full &= ~(uint64_t(1) << j);
      }
#pragma unroll
      for (int j = 0; j < kVecPerLane; ++j) steps = max(steps, last[j] + 1);
      for (int i = 0; i < steps; ++i) {
        // all reads of the step first (the folds below are opaque to the
        // scheduler, so reads placed between them would wait one by one)
        int k[kVecPerLane];
        GridPt q[kVecPerLane];
#pragma unroll
        for (int j = 0; j < kVecPerLane; ++j) k[j] = s_list[at[j] + min(i, last[j])];
#pragma unroll
        for (int j = 0; j < kVecPerLane; ++j) q[j] = s_grid[k[j]];
#pragma unroll
        for (int j = 0; j < kVecPerLane; ++j) fold(j, k[j], q[j]);
      }
    }
    // Vectors that scan every point. Without an index that is every vector:
    // each lane scans for its own, a point read once for all of them. With one
    // it is the few per thousand outside the buckets, one after the
    // other over the whole wave, lane l taking points l, l + 64, ...: a scan by
    // the vector's own lane is a chain of n LDS reads that the rest of the wave
    // waits for (14336 x 4096, 256 points: 247 us against 189; 4096 x 4096, 1024
    // points, g = 256: 268 against 110).
    if (!pruned) {
      const int part = shared ? (n + kQW - 1) / kQW : n;
      const int k0 = shared ? min(wave * part, n) : 0, k1 = min(k0 + part, n);
#pragma unroll 4
      for (int k = k0; k < k1; ++k) {
        const GridPt q = s_grid[k];
#pragma unroll
        for (int j = 0; j < kVecPerLane; ++j) fold(j, k, q);
      }
    } else if (kN <= 16) {  // (a scan is short)
#pragma unroll
      for (int j = 0; j < kVecPerLane; ++j)
        if ((full >> j) & 1)
          for (int k = 0; k < n; ++k) fold(j, k, s_grid[k]);
    } else if (__any(full != 0)) {
#pragma unroll
      for (int j = 0; j < kVecPerLane; ++j) {
        uint64_t todo = __ballot((full >> j) & 1);
        while (todo != 0) {  // uniform
          const int src = __builtin_ctzll(todo);
          todo &= todo - 1;
          double x[P];
#pragma unroll
          for (int t = 0; t < P; ++t) x[t] = readlane_f64(v[j * P + t], src);
          double b = INFINITY;
          for (int k = lane; k < n; k += 64) {
            const GridPt q = s_grid[k];
            double c = fma(-x[0], double(q.x[0]), search_const<P>(q, shift));
            if constexpr (P == 2) c = fma(-x[P - 1], double(q.x[1]), c);
            // (the index differs by lane here)
            const uint64_t u = __builtin_bit_cast(uint64_t, c);
            b = min_f64(b, __builtin_bit_cast(
                               double, (u & ~uint64_t(kIndexMask)) | uint64_t(uint32_t(k))));
          }
          b = wave_min(b, lane);
          if (lane == src) best[j] = b;
        }
      }
    }

    if constexpr (kShare) {
      if (shared) {
        // least over the waves: search values are positive, so their bits are
        // in their order
        unsigned long long* const s_best =
            kInList ? reinterpret_cast<unsigned long long*>(s_list) : s_values;
        if (wave == 0) {
#pragma unroll
          for (int j = 0; j < kVecPerLane; ++j)
            s_best[64 * j + lane] = __builtin_bit_cast(unsigned long long, best[j]);
        }
        __syncthreads();
        if (wave != 0) {
#pragma unroll
          for (int j = 0; j < kVecPerLane; ++j)
            atomicMin(&s_best[64 * j + lane], __builtin_bit_cast(unsigned long long, best[j]));
        }
        __syncthreads();
        // (the others' next use of s_best is behind the barrier that the first
        // wave reaches after this read)
        if (wave != 0) continue;
#pragma unroll
        for (int j = 0; j < kVecPerLane; ++j)
          best[j] = __builtin_bit_cast(double, s_best[64 * j + lane]);
      }
    }

#pragma unroll
    for (int j = 0; j < kVecPerLane; ++j)
      s_codes[code0 + (P == 2 ? fwht_rows_reg<G>(2 * j) >> 1 : fwht_rows_reg<G>(j))] =
          CodeT(__builtin_bit_cast(uint64_t, best[j]) & kIndexMask);
    wave_sync();
    const int64_t grp0 = seg * kSegGroups;
    const int here = groups - grp0 < kSegGroups ? int(groups - grp0) : kSegGroups;
    uint32_t* dst = reinterpret_cast<uint32_t*>(codes) + grp0 * kWordsPerGroup;
    for (int wi = lane; wi < here * kWordsPerGroup; wi += 64) {
      if constexpr (BITS == 8) {  // packed as they are
        dst[wi] = reinterpret_cast<const uint32_t*>(s_codes)[wi];
        continue;
      }
      if constexpr (BITS == 4) {  // eight bytes to eight nibbles
        const uint2 b = reinterpret_cast<const uint2*>(s_codes)[wi];
        const uint32_t x = (b.x | b.x >> 4) & 0x00ff00ffu, y = (b.y | b.y >> 4) & 0x00ff00ffu;
        dst[wi] = ((x | x >> 8) & 0xffffu) | (y | y >> 8) << 16;
        continue;
      }
      const int bit0 = wi * 32;
      int c = bit0 / BITS;
      uint32_t word = uint32_t(s_codes[c]) >> (bit0 - c * BITS);
      for (++c; c * BITS < bit0 + 32 && c < kSegCodes; ++c)
        word |= uint32_t(s_codes[c]) << (c * BITS - bit0);
      dst[wi] = word;
    }
    const int lg = lane / kGroupLanes;
    if (lane % kGroupLanes == 0 && lg < here)
      scales[grp0 + lg] = f64_to_f16_rne(s * inv_sqrt_g);
    wave_sync();
  }
}

// Groups of 2048 and 4096 weights (E = 32, 64): every vector scans all n
// points, the waves of a block step through groups together. The candidate
// walk of quantize_kernel is not used at these sizes: its build for p = 2,
// g = 4096 (32 vectors per lane, registers spilled to the accumulation
// registers) did not finish on the GPU, and the cause has not been found.
template <int E, int P, int BITS, typename InT>
__global__ __launch_bounds__(64 * kWaves) void quantize_scan_kernel(
    const InT* __restrict__ w, int64_t rows, int64_t in, uint64_t seed,
    const float* __restrict__ grid, int n, uint8_t* __restrict__ codes, int64_t row_bytes,
    uint16_t* __restrict__ scales) {
  constexpr int G = 64 * E;
  constexpr int kVecPerLane = E / P;
  constexpr int kCodesPerGroup = G / P;
  constexpr int kWordsPerGroup = kCodesPerGroup * BITS / 32;
  static_assert(E % P == 0, "a lane must hold whole p-vectors");
  static_assert((kCodesPerGroup * BITS) % 32 == 0, "group must fill whole dwords");

  // grid point k: P coordinates then |G_k|^2 / 2 + shift (stride P + 1)
  __shared__ double s_grid[kMaxN * (P + 1)];
  __shared__ uint16_t s_codes[kWaves][kMaxG / P];

  const int lane = int(threadIdx.x) & 63;
  const int wave = int(threadIdx.x) >> 6;

  __shared__ double s_r2[kWaves];
  double r2 = 0.0;  // largest squared grid-point norm seen by this thread
  for (int k = int(threadIdx.x); k < n; k += 64 * kWaves) {
    double h = 0.0;
#pragma unroll
    for (int t = 0; t < P; ++t) {
      const double c = double(grid[k * P + t]);
      s_grid[k * (P + 1) + t] = c;
      h += c * c;
    }
    s_grid[k * (P + 1) + P] = 0.5 * h;
    r2 = fmax(r2, h);
  }
  r2 = wave_max(r2, int(threadIdx.x) & 63);
  if ((threadIdx.x & 63) == 0) s_r2[threadIdx.x >> 6] = r2;
  __syncthreads();
  for (int w = 0; w < kWaves; ++w) r2 = fmax(r2, s_r2[w]);
  // the search-value shift: a power of two at least twice the largest |c_k|
  const double bound = 2.0 * (0.5 * r2 + sqrt(double(64 * E)) * sqrt(r2));
  const double shift = bound <= kMinShift ? kMinShift : exp2(ceil(log2(bound)));
  for (int k = int(threadIdx.x); k < n; k += 64 * kWaves) s_grid[k * (P + 1) + P] += shift;

  uint64_t neg = 0;
#pragma unroll
  for (int i = 0; i < E; ++i) neg |= uint64_t(rht_sign_negative(seed, uint32_t(lane * E + i))) << i;

  const int64_t groups_per_row = in / G;
  const int64_t total = rows * groups_per_row;
  const double inv_sqrt_g = 1.0 / sqrt(double(G));
  __syncthreads();

  // Every wave of the block runs the same number of iterations (barriers).
  for (int64_t first = int64_t(blockIdx.x) * kWaves; first < total;
       first += int64_t(gridDim.x) * kWaves) {
    const int64_t grp = first + wave;
    const bool valid = grp < total;
    const int64_t row = valid ? grp / groups_per_row : 0;
    const int64_t gi = valid ? grp - row * groups_per_row : 0;

    double v[E];
    if (valid) {
      load_group<E, InT>(w + row * in + gi * G + lane * E, v);
    } else {
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = 0.0;
    }

    double ss = 0.0;
#pragma unroll
    for (int i = 0; i < E; ++i) ss += v[i] * v[i];
    ss = wave_sum(ss, lane);
    const double s = sqrt(ss);

#pragma unroll
    for (int i = 0; i < E; ++i) {
      const double u = s > 0.0 ? v[i] / s : 0.0;
      v[i] = ((neg >> i) & 1) ? -u : u;
    }
    fwht_wave<E>(v, lane, G);

    double best[kVecPerLane];
#pragma unroll
    for (int j = 0; j < kVecPerLane; ++j) best[j] = INFINITY;
    const uint32_t index_mask = kIndexMask;
    for (int k = 0; k < n; ++k) {
      double gk[P];
#pragma unroll
      for (int t = 0; t < P; ++t) gk[t] = s_grid[k * (P + 1) + t];
      const double hk = s_grid[k * (P + 1) + P];
#pragma unroll
      for (int j = 0; j < kVecPerLane; ++j) {
        double c = hk;
#pragma unroll
        for (int t = 0; t < P; ++t) c = fma(-v[j * P + t], gk[t], c);
        best[j] = min_indexed(best[j], c, uint32_t(k), index_mask);
      }
    }

#pragma unroll
    for (int j = 0; j < kVecPerLane; ++j)
      s_codes[wave][lane * kVecPerLane + j] =
          uint16_t(__builtin_bit_cast(uint64_t, best[j]) & kIndexMask);
    __syncthreads();

    if (valid) {
      uint32_t* dst = reinterpret_cast<uint32_t*>(codes + row * row_bytes +
                                                  gi * (int64_t(kCodesPerGroup) * BITS / 8));
      for (int wi = lane; wi < kWordsPerGroup; wi += 64) {
        const int bit0 = wi * 32;
        int c = bit0 / BITS;
        uint32_t word = uint32_t(s_codes[wave][c]) >> (bit0 - c * BITS);
        for (++c; c * BITS < bit0 + 32 && c < kCodesPerGroup; ++c)
          word |= uint32_t(s_codes[wave][c]) << (c * BITS - bit0);
        dst[wi] = word;
      }
      if (lane == 0) scales[row * groups_per_row + gi] = f64_to_f16_rne(s * inv_sqrt_g);
    }
    __syncthreads();
  }
}


// Little-endian dword at any byte address.
struct __attribute__((packed, aligned(1))) AnyU32 {
  uint32_t v;
};

// Quantization error of a layer, measured in the rotated space: the rotation
// R = H diag(sigma) / sqrt(g) is orthonormal, so per group (Parseval)
//   ||w - w_hat||^2 = || H (sigma * w) / sqrt(g) - scale * concat_j G[code_j] ||^2
// with w_hat the dequantised group (App. G). One wavefront per group writes
// that sum and ||w||^2 as two fp64 values (row-major group order); the layer's
// relative error t^2 (Sec. 3.4) is their ratio of sums. The group's codes are
// read as whole dwords into the wave's LDS and the grid is kept in LDS: read
// from memory per code (three bytes and a gather each), the vector memory
// unit was the bound (4096 x 14336 bf16, 6-bit codes: 152 us; 100 us with both
// in LDS, 64 us with the rotation through LDS for g = 1024 and the next group's
// loads issued ahead). Now bound by the vector ALU: about 450 instructions per
// 1024 weights and lane, two thirds of them fp64.
template <int E, int P, int BITS, typename InT>
__global__ __launch_bounds__(64 * kWaves) void layer_error_kernel(
    const InT* __restrict__ w, int64_t rows, int64_t in, uint64_t seed,
    const float* __restrict__ grid, const uint8_t* __restrict__ codes,
    const uint16_t* __restrict__ scales, double* __restrict__ out) {
  constexpr int G = 64 * E;
  constexpr int V = E / P;                      // codes per lane
  constexpr int kWords = G / P * BITS / 32;     // dwords of a group's codes
  constexpr int kLaneWords = (V * BITS + 31) / 32;
  static_assert(E % P == 0, "a lane must hold whole p-vectors");
  static_assert(G / P * BITS % 32 == 0, "group must fill whole dwords");
  // g = 1024: rotated through LDS, which leaves a lane other elements than it
  // read; the unpacked codes go through LDS as well
  constexpr bool kRows = E == 16;
  // small grids are kept in fp64 (no conversion per element)
  using GridT = typename std::conditional<((P << BITS) <= 512), double, float>::type;
  __shared__ GridT s_grid[P << BITS];
  __shared__ uint32_t s_words[kWaves][kWords + 2];  // a lane's window may end past its codes
  __shared__ __align__(16) uint32_t s_rot[kWaves][kRows ? kFwhtRows : 4];
  __shared__ __align__(16) uint16_t s_code[kWaves][kRows ? G / P : 8];
  __shared__ uint64_t s_neg[E];
  const int lane = int(threadIdx.x) & 63;
  const int wave = int(threadIdx.x) >> 6;
  for (int k = int(threadIdx.x); k < P << BITS; k += 64 * kWaves) s_grid[k] = GridT(grid[k]);
  if (lane < 2) s_words[wave][kWords + lane] = 0;
  block_signs<E, kWaves>(seed, s_neg, wave, lane);
  uint32_t flips[RawGroup<E, InT>::kMasks];
  RawGroup<E, InT>::masks(s_neg[lane * E / 64] >> (lane * E % 64), flips);
  // groups, their scales and their codes all lie back to back
  const int64_t total = rows * (in / G);
  const double inv_sqrt_g = 1.0 / sqrt(double(G));
  const int bit0 = lane * V * BITS;
  const uint32_t* mine = &s_words[wave][bit0 >> 5];
  const int n0 = fwht_rows_lane<1024>(lane);
  // what a group needs from memory, requested one group ahead
  RawGroup<E, InT> raw;
  uint32_t cd[(kWords + 63) / 64];
  uint16_t sc = 0;
  auto request = [&](int64_t grp) {
    raw.load(w + grp * G + lane * E);
    const AnyU32* cw = reinterpret_cast<const AnyU32*>(codes) + grp * kWords;
#pragma unroll
    for (int q = 0; q < (kWords + 63) / 64; ++q)
      cd[q] = 64 * q + lane < kWords ? cw[64 * q + lane].v : 0u;
    sc = scales[grp];
  };
  // no barrier below: each wave walks its own groups
  const int64_t step = int64_t(gridDim.x) * kWaves;
  int64_t grp = int64_t(blockIdx.x) * kWaves + wave;
  if (grp < total) request(grp);
  for (; grp < total; grp += step) {
    const double sh = double(__builtin_bit_cast(_Float16, sc));
    double v[E];
    raw.flip(flips);  // sigma
    raw.expand(v);
    wave_sync();  // the last group's words have been read
#pragma unroll
    for (int q = 0; q < (kWords + 63) / 64; ++q)
      if (64 * q + lane < kWords) s_words[wave][64 * q + lane] = cd[q];
    wave_sync();
    if (grp + step < total) request(grp + step);
    // the lane's codes: of its own vectors
    uint32_t win[kLaneWords], code[V];
#pragma unroll
    for (int q = 0; q < kLaneWords; ++q)
      win[q] = __builtin_amdgcn_alignbit(mine[q + 1], mine[q], uint32_t(bit0 & 31));
#pragma unroll
    for (int t = 0; t < V; ++t) {
      const int b = t * BITS, wq = b >> 5, o = b & 31;
      uint32_t c = win[wq] >> o;
      if (o + BITS > 32) c |= win[wq + 1 < kLaneWords ? wq + 1 : wq] << (32 - o);
      code[t] = c & ((1u << BITS) - 1u);
    }
    if constexpr (kRows) {
      u32x4* dst = reinterpret_cast<u32x4*>(&s_code[wave][lane * V]);
#pragma unroll
      for (int q = 0; q < V / 8; ++q)
        dst[q] = u32x4{code[8 * q] | code[8 * q + 1] << 16, code[8 * q + 2] | code[8 * q + 3] << 16,
                       code[8 * q + 4] | code[8 * q + 5] << 16,
                       code[8 * q + 6] | code[8 * q + 7] << 16};
    }
    double ss = 0.0;
#pragma unroll
    for (int i = 0; i < E; ++i) ss += v[i] * v[i];
    ss = wave_sum(ss, lane);
    double e = 0.0;
    if constexpr (kRows) {
      fwht_rows<1024>(v, s_rot[wave], lane);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int n = n0 + fwht_rows_reg<1024>(r);
        const uint32_t c = s_code[wave][n / P];
        // in units of 1 / sqrt(g) = 1 / 32: exact, one multiply less
        const double d = fma(-32.0 * sh, double(s_grid[c * P + (n & (P - 1))]), v[r]);
        e += d * d;
      }
      e *= inv_sqrt_g * inv_sqrt_g;
    } else {
      fwht_wave<E>(v, lane, G);
#pragma unroll
      for (int t = 0; t < V; ++t)
#pragma unroll
        for (int c = 0; c < P; ++c) {
          const double d = v[t * P + c] * inv_sqrt_g - sh * double(s_grid[code[t] * P + c]);
          e += d * d;
        }
    }
    e = wave_sum(e, lane);
    if (lane == 0) {
      out[2 * grp] = e;
      out[2 * grp + 1] = ss;
    }
  }
}

// t^2 = sum_q err_q / sum_q norm_q over the per-group pairs of
// layer_error_kernel (Sec. 3.4's relative error of the layer). One block (no
// memory for partial sums here): thread t adds the pairs t, t + 1024, ... in
// order, sixteen loads in flight, then a fixed tree over the threads
// (deterministic). A layer of norm 0 gets t^2 = 0. Bound by one compute unit's
// loads: 57344 groups take 12 us (57 us with 256 threads and one load at a time).
__global__ __launch_bounds__(1024) void layer_t2_kernel(const double* __restrict__ pairs,
                                                        int64_t groups, double* __restrict__ t2) {
  __shared__ double s_e[1024], s_n[1024];
  const int tid = int(threadIdx.x);
  double e = 0.0, nrm = 0.0;
  constexpr int kAhead = 16;
  for (int64_t q0 = tid; q0 < groups; q0 += 1024 * kAhead) {
    double pe[kAhead], pn[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const int64_t q = q0 + 1024 * i;
      const int64_t at = q < groups ? q : q0;
      pe[i] = pairs[2 * at];
      pn[i] = pairs[2 * at + 1];
    }
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if (q0 + 1024 * i < groups) {
        e += pe[i];
        nrm += pn[i];
      }
  }
  s_e[tid] = e;
  s_n[tid] = nrm;
  __syncthreads();
  for (int h = 512; h > 0; h >>= 1) {
    if (tid < h) {
      s_e[tid] += s_e[tid + h];
      s_n[tid] += s_n[tid + h];
    }
    __syncthreads();
  }
  if (tid == 0) t2[0] = s_n[0] > 0.0 ? s_e[0] / s_n[0] : 0.0;
}

template <int P, int BITS, typename InT>
hipError_t launch_error_p(const InT* w, int64_t out_rows, int64_t in, const float* grid, int g,
                          uint64_t seed, const uint8_t* codes, const uint16_t* scales,
                          double* err, hipStream_t stream) {
  const int64_t total = out_rows * (in / g);
  // eight blocks per compute unit: a block reads the grid and forms the signs
  // once, then its waves take groups in turn
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((total + kWaves - 1) / kWaves, 2048));
  const dim3 grid_dim{unsigned(blocks)}, block{64 * kWaves};
  switch (g) {
#define HIGGS_E_CASE(GV)                                                                     \
  case GV:                                                                                   \
    if constexpr ((GV / 64) % P == 0) {                                                      \
      hipLaunchKernelGGL((layer_error_kernel<GV / 64, P, BITS, InT>), grid_dim, block, 0,    \
                         stream, w, out_rows, in, seed, grid, codes, scales, err);           \
      return hipGetLastError();                                                              \
    }                                                                                        \
    break;
    HIGGS_E_CASE(64)
    HIGGS_E_CASE(128)
    HIGGS_E_CASE(256)
    HIGGS_E_CASE(512)
    HIGGS_E_CASE(1024)
    HIGGS_E_CASE(2048)
    HIGGS_E_CASE(4096)
#undef HIGGS_E_CASE
    default:
      break;
  }
  return hipErrorInvalidValue;
}

template <typename InT>
hipError_t launch_error_typed(const InT* w, int64_t out, int64_t in, const float* grid, int p,
                              int bits, int g, uint64_t seed, const uint8_t* codes,
                              const uint16_t* scales, double* err, hipStream_t stream) {
#define HIGGS_E_FORMAT(PV, BV)                                                              \
  if (p == PV && bits == BV)                                                                \
    return launch_error_p<PV, BV>(w, out, in, grid, g, seed, codes, scales, err, stream);
  HIGGS_E_FORMAT(1, 4)
  HIGGS_E_FORMAT(1, 8)
  HIGGS_E_FORMAT(2, 6)
  HIGGS_E_FORMAT(2, 8)
  HIGGS_E_FORMAT(2, 10)
#undef HIGGS_E_FORMAT
  return hipErrorInvalidValue;
}

template <int P, int BITS, typename InT>
hipError_t launch_bits(const InT* w, int64_t out, int64_t in, const float* grid, int n,
                       const uint8_t* index, int g, uint64_t seed, uint8_t* codes,
                       int64_t row_bytes, uint16_t* scales, hipStream_t stream) {
  const int64_t total = out * (in / g);
  // a block loads the grid and the index into LDS once, then its waves take
  // 1024 weights at a time. The 256- and 1024-point grids' indexes nearly fill
  // a compute unit's LDS, and scalar grids run 2 waves per SIMD (registers):
  // there one block per compute unit with 12 or 8 waves; else blocks of 4
  // waves, up to 2048 (measured faster there)
  constexpr int kQW = P == 1 ? 8 : (BITS >= 8 ? 12 : 4);
  constexpr int64_t kMaxBlocks = kQW == 4 ? 2048 : 256;
  const int64_t segs = (total + std::max(1, 1024 / g) - 1) / std::max(1, 1024 / g);
  // no index and weights for at most half the compute units: the waves of a
  // block share 1024 weights (quantize_kernel)
  const bool shared = index == nullptr && BITS > 4 && segs <= 128 * kQW;
  const int64_t blocks = std::max<int64_t>(
      1, std::min<int64_t>(shared ? segs : (segs + kQW - 1) / kQW, kMaxBlocks));
  const dim3 grid_dim{unsigned(blocks)}, block{64 * kQW}, scan_block{64 * kWaves};
  switch (g) {
#define HIGGS_Q_CASE(GV)                                                                     \
  case GV:                                                                                   \
    if constexpr (GV >= 64 * P) {                                                            \
      hipLaunchKernelGGL((quantize_kernel<GV, P, BITS, kQW, InT>), grid_dim, block, 0,       \
                         stream, w, total, seed, grid, n, index, shared, codes, scales);     \
      return hipGetLastError();                                                              \
    }                                                                                        \
    break;
    HIGGS_Q_CASE(64)
    HIGGS_Q_CASE(128)
    HIGGS_Q_CASE(256)
    HIGGS_Q_CASE(512)
    HIGGS_Q_CASE(1024)
#undef HIGGS_Q_CASE
    default:
      break;
  }
  // larger groups: the full scan, one block per four groups
  const dim3 scan_grid{unsigned(std::min<int64_t>((total + kWaves - 1) / kWaves, 8192))};
  switch (g) {
#define HIGGS_S_CASE(GV)                                                                     \
  case GV:                                                                                   \
    if constexpr ((GV / 64) % P == 0) {                                                      \
      hipLaunchKernelGGL((quantize_scan_kernel<GV / 64, P, BITS, InT>), scan_grid,           \
                         scan_block, 0, stream, w, out, in, seed, grid, n, codes, row_bytes, \
                         scales);                                                            \
      return hipGetLastError();                                                              \
    }                                                                                        \
    break;
    HIGGS_S_CASE(2048)
    HIGGS_S_CASE(4096)
#undef HIGGS_S_CASE
    default:
      break;
  }
  return hipErrorInvalidValue;
}

template <typename InT>
hipError_t launch_typed(const InT* w, int64_t out, int64_t in, const float* grid, int p, int n,
                        const uint8_t* index, int g, uint64_t seed, uint8_t* codes,
                        uint16_t* scales, hipStream_t stream) {
  const int bits = code_bits(p, n);
  const int64_t row_bytes = in / p * bits / 8;
  if (p == 1 && bits == 4)
    return launch_bits<1, 4>(w, out, in, grid, n, index, g, seed, codes, row_bytes,
                             scales, stream);
  if (p == 1 && bits == 8)
    return launch_bits<1, 8>(w, out, in, grid, n, index, g, seed, codes, row_bytes,
                             scales, stream);
  if (p == 2 && bits == 6)
    return launch_bits<2, 6>(w, out, in, grid, n, index, g, seed, codes, row_bytes,
                             scales, stream);
  if (p == 2 && bits == 8)
    return launch_bits<2, 8>(w, out, in, grid, n, index, g, seed, codes, row_bytes,
                             scales, stream);
  if (p == 2 && bits == 10)
    return launch_bits<2, 10>(w, out, in, grid, n, index, g, seed, codes, row_bytes,
                              scales, stream);
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// GPTQ rounding in place of the nearest-point step (Sec. 3.5), in the rotated
// space: W' = per group H (sigma * w) / sqrt(g), the Hessian of the rotated
// calibration activations, U the upper Cholesky factor of its damped inverse
// (Hinv = U^T U). Columns are taken in order, one p-vector at a time: its
// rotated weights v are rounded like Alg. 1 (nearest grid point of
// v sqrt(g) / s, s the group's norm), the error e = v - (s / sqrt(g)) G[q] is
// scaled, E = e U_pp^-1 (U_pp the p x p diagonal block), and later columns
// move by -E U[p-vector, later]. Within a block of 64 columns the update runs
// here; E takes the place of the block's columns of W', and later columns get
// their updates from it by matrix products (gptq.cpp).
// ---------------------------------------------------------------------------

// Rotated weights W' (fp64), each group's norm s (fp64) and the stored scale
// fp16(s / sqrt(g)). One wavefront per group.
template <int E, typename InT>
__global__ __launch_bounds__(64 * kWaves) void gptq_prepare_kernel(
    const InT* __restrict__ w, int64_t rows, int64_t in, uint64_t seed, double* __restrict__ wr,
    double* __restrict__ norms, uint16_t* __restrict__ scales) {
  constexpr int G = 64 * E;
  constexpr bool kRows = E == 16;  // g = 1024: rotated through LDS
  __shared__ __align__(16) uint32_t s_rot[kWaves][kRows ? kFwhtRows : 4];
  __shared__ uint64_t s_neg[E];
  const int lane = int(threadIdx.x) & 63;
  const int wave = int(threadIdx.x) >> 6;
  block_signs<E, kWaves>(seed, s_neg, wave, lane);
  const uint64_t neg = s_neg[lane * E / 64] >> (lane * E % 64);
  const int64_t total = rows * (in / G);  // groups lie back to back
  const double inv_sqrt_g = 1.0 / sqrt(double(G));
  for (int64_t grp = int64_t(blockIdx.x) * kWaves + wave; grp < total;
       grp += int64_t(gridDim.x) * kWaves) {
    double v[E];
    load_group<E, InT>(w + grp * G + lane * E, v);
    double ss = 0.0;
#pragma unroll
    for (int i = 0; i < E; ++i) ss += v[i] * v[i];
    ss = wave_sum(ss, lane);
    const double sn = sqrt(ss);
#pragma unroll
    for (int i = 0; i < E; ++i)
      if ((neg >> i) & 1) v[i] = -v[i];
    double* dst = wr + grp * G;
    if constexpr (kRows) {
      fwht_rows<1024>(v, s_rot[wave], lane);
#pragma unroll
      for (int i = 0; i < E; ++i)
        dst[fwht_rows_lane<1024>(lane) + fwht_rows_reg<1024>(i)] = v[i] * inv_sqrt_g;
    } else {
      fwht_wave<E>(v, lane, G);
#pragma unroll
      for (int i = 0; i < E; ++i) dst[lane * E + i] = v[i] * inv_sqrt_g;
    }
    if (lane == 0) {
      norms[grp] = sn;
      scales[grp] = f64_to_f16_rne(sn * inv_sqrt_g);
    }
  }
}

// The value of lane L of this lane's row of 16 lanes.
template <int L>
__device__ inline double row16_lane(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo =
      uint32_t(__builtin_amdgcn_mov_dpp(int(uint32_t(u)), 0x150 + L, 0xF, 0xF, true));
  const uint32_t hi =
      uint32_t(__builtin_amdgcn_mov_dpp(int(uint32_t(u >> 32)), 0x150 + L, 0xF, 0xF, true));
  return __builtin_bit_cast(double, uint64_t(lo) | (uint64_t(hi) << 32));
}

// f(0), f(1), ..., f(N - 1) with compile-time arguments.
template <int N, int I = 0, typename F>
__device__ __attribute__((always_inline)) inline void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// One block of 64 columns [c0, c0 + 64) for every row of W'. LPR lanes share a
// row of W' (16, 32 or 64 for grids of 16, up to 256, and 1024 points): lane s
// of them holds the grid points s, s + LPR, ... (16 at most) in registers, and
// each of their 16-lane rows holds all 64 columns (lane c: columns c, c + 16,
// ...), so that a column's value reaches every lane by one DPP broadcast. The
// p-vectors of a row are a serial chain, and a layer has few rows for a chip,
// so the chain's length is the time: per p-vector the broadcast, the lane's
// candidates (two fma and a minimum each), a minimum over the row's lanes, the
// lowest index that has it, the error, and the later columns' update. 32 lanes
// per row give 4096 rows two wavefronts per SIMD, which hide each other's
// latencies (16 lanes, one wavefront: 36 us per block of columns; 32 lanes: 24
// us; a wavefront per row with the candidates in LDS and the minimum found by
// LDS shuffles of (value, index): 90 us). Quotients by U's diagonal are formed
// from its reciprocals with one correction step.
constexpr int kGptqWaves = 8;

template <int P, int N>
__global__ __launch_bounds__(64 * kGptqWaves, 2) void gptq_block_kernel(
    double* __restrict__ wr, const double* __restrict__ norms, const double* __restrict__ u,
    const float* __restrict__ grid, int64_t rows, int64_t in, int log2g, int64_t c0,
    uint8_t* __restrict__ codes, int64_t row_bytes) {
  constexpr int kB = 64;
  constexpr int kBits = N == 16 ? 4 : N == 64 ? 6 : N == 256 ? 8 : 10;
  constexpr int LPR = N > 256 ? 64 : N > 16 ? 32 : 16;
  constexpr int kRowsPerWave = 64 / LPR;
  constexpr int KC = kB / 16;                  // columns per lane
  constexpr int kCand = N / LPR;               // grid points per lane
  constexpr int kVecs = kB / P;
  constexpr int kWordsPerRow = kVecs * kBits / 32;
  static_assert(kWordsPerRow <= LPR, "one lane per packed dword");
  __shared__ double s_u[kB][kB];
  __shared__ double s_r[kB];                   // 1 / U's diagonal
  __shared__ double s_grid[N * P];
  __shared__ uint16_t s_codes[kGptqWaves * kRowsPerWave][kVecs];
  const int tid = int(threadIdx.x);
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int sub = lane % LPR;  // candidates sub, sub + LPR, ...
  const int col = lane & 15;   // columns col, col + 16, ...
  const int rslot = wave * kRowsPerWave + lane / LPR;
  for (int i = tid; i < kB * kB; i += 64 * kGptqWaves) {
    const int r = i / kB, c = i % kB;
    const double x = c >= r ? u[(c0 + r) * in + c0 + c] : 0.0;  // upper triangle only
    s_u[r][c] = x;
    if (r == c) s_r[r] = 1.0 / x;
  }
  for (int k = tid; k < N * P; k += 64 * kGptqWaves) s_grid[k] = double(grid[k]);
  __syncthreads();
  const int64_t row_id = int64_t(blockIdx.x) * (kGptqWaves * kRowsPerWave) + rslot;
  const bool valid = row_id < rows;            // rows past the end repeat the last one
  const int64_t row = valid ? row_id : rows - 1;
  // the lane's candidates: coordinates and |G|^2 / 2
  double cg[kCand][P], ch[kCand];
#pragma unroll
  for (int j = 0; j < kCand; ++j) {
    double h = 0.0;
#pragma unroll
    for (int d = 0; d < P; ++d) {
      cg[j][d] = s_grid[(sub + LPR * j) * P + d];
      h += cg[j][d] * cg[j][d];
    }
    ch[j] = 0.5 * h;
  }
  const int g = 1 << log2g;
  const double sn = norms[row * (in >> log2g) + (c0 >> log2g)];  // the block is in one group
  const double fwd = sn > 0.0 ? sqrt(double(g)) / sn : 0.0;      // W' -> grid units
  const double back = sn / sqrt(double(g));                      // grid units -> W'
  double* wrow = wr + row * in + c0;
  double wv[KC];
#pragma unroll
  for (int k = 0; k < KC; ++k) wv[k] = wrow[col + 16 * k];
  // columns 16 k .. 16 k + 15 are in wv[0] at turn k
  for (int k = 0; k < KC; ++k) {
    double my_err = 0.0;
    uint32_t my_q = 0;
    const double* uk = &s_u[16 * k][16 * k];  // row 16 k, from column 16 k on
    static_for<16 / P>([&](auto T) __attribute__((always_inline)) {
      constexpr int i0 = decltype(T)::value * P;  // column inside the turn
      double v[P], uv[P];
      static_for<P>([&](auto D) __attribute__((always_inline)) {
        constexpr int d = decltype(D)::value;
        v[d] = row16_lane<i0 + d>(wv[0]);
        uv[d] = v[d] * fwd;
      });
      // nearest grid point, the lowest index on ties: the least value over the
      // lane's candidates and the row's lanes, then the least index that has it
      double c[kCand], best;
#pragma unroll
      for (int j = 0; j < kCand; ++j) {
        c[j] = ch[j];
#pragma unroll
        for (int d = 0; d < P; ++d) c[j] = fma(-uv[d], cg[j][d], c[j]);
      }
      double m[kCand];
#pragma unroll
      for (int j = 0; j < kCand; ++j) m[j] = c[j];
#pragma unroll
      for (int h = kCand / 2; h > 0; h >>= 1)
#pragma unroll
        for (int j = 0; j < h; ++j) m[j] = min_f64(m[j], m[j + h]);
      best = m[0];
      best = min_f64(best, lane_xor<1>(best, lane));
      best = min_f64(best, lane_xor<2>(best, lane));
      best = min_f64(best, lane_xor<4>(best, lane));
      best = min_f64(best, lane_xor<8>(best, lane));
      if constexpr (LPR >= 32) best = min_f64(best, lane_xor<16>(best, lane));
      if constexpr (LPR == 64) best = min_f64(best, lane_xor<32>(best, lane));
      uint32_t q = N;
#pragma unroll
      for (int j = kCand - 1; j >= 0; --j) q = c[j] == best ? uint32_t(sub + LPR * j) : q;
      q = min(q, lane_xor_u32<1>(q, lane));
      q = min(q, lane_xor_u32<2>(q, lane));
      q = min(q, lane_xor_u32<4>(q, lane));
      q = min(q, lane_xor_u32<8>(q, lane));
      if constexpr (LPR >= 32) q = min(q, lane_xor_u32<16>(q, lane));
      if constexpr (LPR == 64) q = min(q, lane_xor_u32<32>(q, lane));
      q = q < N ? q : 0;  // (no value compares equal: NaN)
      double e[P], es[P];
#pragma unroll
      for (int d = 0; d < P; ++d) e[d] = v[d] - back * s_grid[q * P + d];
      // E = e U_pp^-1 (U_pp upper triangular)
      const double* u0 = uk + i0 * (kB + 1);  // U's diagonal at the p-vector
#pragma unroll
      for (int d = 0; d < P; ++d) {
        double num = e[d];
        if (d > 0) num = e[d] - es[0] * u0[1];
        const double rd = s_r[16 * k + i0 + d], ud = u0[d * (kB + 1)];
        const double q0 = num * rd;
        es[d] = fma(fma(-q0, ud, num), rd, q0);
      }
      // later columns (U is zero below its diagonal; the p-vector's own
      // columns are done with)
#pragma unroll
      for (int j = 0; j < KC; ++j) {
        const int cj = min(col + 16 * j, kB - 1 - 16 * k);  // past the block: unused
#pragma unroll
        for (int d = 0; d < P; ++d) wv[j] = fma(-es[d], uk[(i0 + d) * kB + cj], wv[j]);
      }
#pragma unroll
      for (int d = 0; d < P; ++d)
        my_err = col == i0 + d ? es[d] : my_err;
      my_q = col == i0 / P ? q : my_q;  // lane t of a row keeps the turn's t-th code
    });
    if (valid && sub < 16) wrow[16 * k + col] = my_err;
    if (sub < 16 / P) s_codes[rslot][16 / P * k + sub] = uint16_t(my_q);
#pragma unroll
    for (int j = 0; j + 1 < KC; ++j) wv[j] = wv[j + 1];
  }
  wave_sync();
  // pack the block's codes: whole dwords
  uint32_t* dst = reinterpret_cast<uint32_t*>(codes + row * row_bytes + (c0 / P) * kBits / 8);
  if (valid && sub < kWordsPerRow) {
    const int bit0 = sub * 32;
    int c = bit0 / kBits;
    uint32_t word = uint32_t(s_codes[rslot][c]) >> (bit0 - c * kBits);
    for (++c; c * kBits < bit0 + 32 && c < kVecs; ++c)
      word |= uint32_t(s_codes[rslot][c]) << (c * kBits - bit0);
    dst[sub] = word;
  }
}

__global__ void f32_to_f64_kernel(const float* __restrict__ src, int64_t count,
                                  double* __restrict__ dst) {
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < count;
       i += int64_t(gridDim.x) * 256)
    dst[i] = double(src[i]);
}

// h[i][i] += damp * mean_i h[i][i] (one block; the mean is summed in a fixed
// order: each thread a strided partial, then thread 0 over the partials)
__global__ __launch_bounds__(256) void damp_diag_kernel(double* __restrict__ h, int64_t in,
                                                        double damp) {
  __shared__ double s_part[256];
  double sum = 0.0;
  for (int64_t i = threadIdx.x; i < in; i += 256) sum += h[i * in + i];
  s_part[threadIdx.x] = sum;
  __syncthreads();
  __shared__ double s_add;
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int k = 0; k < 256; ++k) t += s_part[k];
    s_add = damp * t / double(in);
  }
  __syncthreads();
  for (int64_t i = threadIdx.x; i < in; i += 256) h[i * in + i] += s_add;
}

}  // namespace

hipError_t launch_gptq_prepare(const void* w, higgs_dtype dtype, int64_t out, int64_t in, int g,
                               uint64_t seed, double* wr, double* norms, uint16_t* scales,
                               hipStream_t stream) {
  const int64_t total = out * (in / g);
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((total + kWaves - 1) / kWaves, 8192));
  switch (g) {
#define HIGGS_G_CASE(GV)                                                                        \
  case GV:                                                                                      \
    if (dtype == HIGGS_F32)                                                                     \
      hipLaunchKernelGGL((gptq_prepare_kernel<GV / 64, float>), dim3(unsigned(blocks)),        \
                         dim3(64 * kWaves), 0, stream, static_cast<const float*>(w), out, in,  \
                         seed, wr, norms, scales);                                              \
    else                                                                                        \
      hipLaunchKernelGGL((gptq_prepare_kernel<GV / 64, uint16_t>), dim3(unsigned(blocks)),     \
                         dim3(64 * kWaves), 0, stream, static_cast<const uint16_t*>(w), out,   \
                         in, seed, wr, norms, scales);                                          \
    return hipGetLastError();
    HIGGS_G_CASE(64)
    HIGGS_G_CASE(128)
    HIGGS_G_CASE(256)
    HIGGS_G_CASE(512)
    HIGGS_G_CASE(1024)
    HIGGS_G_CASE(2048)
    HIGGS_G_CASE(4096)
#undef HIGGS_G_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_gptq_block(double* wr, const double* norms, const double* u, const float* grid,
                             int p, int n, int64_t out, int64_t in, int g, int64_t c0,
                             uint8_t* codes, hipStream_t stream) {
  const int64_t row_bytes = in / p * code_bits(p, n) / 8;
#define HIGGS_B_CASE(PV, NV)                                                                    \
  if (p == PV && n == NV) {                                                                     \
    constexpr int kRowsPerBlock = kGptqWaves * (NV > 256 ? 1 : NV > 16 ? 2 : 4);                \
    hipLaunchKernelGGL((gptq_block_kernel<PV, NV>),                                             \
                       dim3(unsigned((out + kRowsPerBlock - 1) / kRowsPerBlock)),               \
                       dim3(64 * kGptqWaves), 0, stream, wr, norms, u, grid, out, in,           \
                       log2_exact(g), c0, codes, row_bytes);                                    \
    return hipGetLastError();                                                                   \
  }
  HIGGS_B_CASE(1, 16)
  HIGGS_B_CASE(1, 256)
  HIGGS_B_CASE(2, 64)
  HIGGS_B_CASE(2, 256)
  HIGGS_B_CASE(2, 1024)
#undef HIGGS_B_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_to_f64(const float* src, int64_t count, double* dst, hipStream_t stream) {
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((count + 255) / 256, 8192));
  hipLaunchKernelGGL(f32_to_f64_kernel, dim3(unsigned(blocks)), dim3(256), 0, stream, src, count,
                     dst);
  return hipGetLastError();
}

hipError_t launch_damp_diag(double* h, int64_t in, double damp, hipStream_t stream) {
  hipLaunchKernelGGL(damp_diag_kernel, dim3(1), dim3(256), 0, stream, h, in, damp);
  return hipGetLastError();
}

hipError_t launch_layer_error(const void* w, higgs_dtype dtype, int64_t out, int64_t in,
                              const uint8_t* codes, const uint16_t* scales, const float* grid,
                              int p, int n, int g, uint64_t seed, double* err, double* t2,
                              hipStream_t stream) {
  const int bits = code_bits(p, n);
  const hipError_t st =
      dtype == HIGGS_F32
          ? launch_error_typed(static_cast<const float*>(w), out, in, grid, p, bits, g, seed,
                               codes, scales, err, stream)
          : launch_error_typed(static_cast<const uint16_t*>(w), out, in, grid, p, bits, g, seed,
                               codes, scales, err, stream);
  if (st != hipSuccess || t2 == nullptr) return st;
  hipLaunchKernelGGL(layer_t2_kernel, dim3(1), dim3(1024), 0, stream, err, out * (in / g), t2);
  return hipGetLastError();
}

hipError_t launch_quantize(const void* w, higgs_dtype dtype, int64_t out, int64_t in,
                           const float* grid, int p, int n, const void* index, int g,
                           uint64_t seed, uint8_t* codes, uint16_t* scales, hipStream_t stream) {
  const uint8_t* idx = static_cast<const uint8_t*>(index);
  if (dtype == HIGGS_F32)
    return launch_typed(static_cast<const float*>(w), out, in, grid, p, n, idx, g, seed, codes,
                        scales, stream);
  return launch_typed(static_cast<const uint16_t*>(w), out, in, grid, p, n, idx, g, seed, codes,
                      scales, stream);
}

int64_t search_index_bytes(int p, int n) { return index_layout(p, n).bytes; }

hipError_t launch_search_index(const float* grid, int p, int n, void* index, hipStream_t stream) {
  uint8_t* idx = static_cast<uint8_t*>(index);
  const dim3 slots_grid{unsigned((index_cells(p, n) + 3) / 4)}, slots_block{256};
#define HIGGS_I_CASE(PV, NV)                                                                 \
  if (p == PV && n == NV) {                                                                  \
    hipLaunchKernelGGL((index_slots_kernel<PV, NV>), slots_grid, slots_block, 0, stream, grid, \
                       n, idx);                                                              \
    hipLaunchKernelGGL((index_finish_kernel<PV, NV>), dim3(1), dim3(1024), 0, stream, grid, n, \
                       idx);                                                                 \
    return hipGetLastError();                                                                \
  }
  HIGGS_I_CASE(1, 16)
  HIGGS_I_CASE(1, 256)
  HIGGS_I_CASE(2, 64)
  HIGGS_I_CASE(2, 256)
  HIGGS_I_CASE(2, 1024)
#undef HIGGS_I_CASE
  return hipErrorInvalidValue;
}

}  // namespace higgs
