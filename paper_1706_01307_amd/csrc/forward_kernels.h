// Forward multiply-add kernels of SC / VSC on gfx950 (Section 4 of the paper: zero
// the output, then for every offset i and pair j add input row R_i(j,1)
// times W^i into output row R_i(j,2); Table 1: a*m*n multiply-adds per active
// output site).
//
// The kernels are output-stationary: a workgroup owns a tile of output rows
// (consecutive positions of the rule book's Z-order schedule, so the tile is
// spatially compact) and keeps their fp32 accumulators in registers while it
// walks the offsets in ascending order.  For offset i it gathers the input
// rows G[i][p] of its positions (the gather map built with the rule book;
// 1 + input row, 0 = no active input, read as zeros) and multiplies them by
// W^i.  Every output element is written once, by one lane, after a
// fixed-order sum: no atomics, bitwise reproducible.
//
//   k_fwd_mfma  dense contraction on the matrix cores: v_mfma 16x16x32 bf16
//               or 16x16x4 f32.  W^i is staged into LDS transposed (one row
//               per output column, XOR-swizzled chunks) and double-buffered
//               across offsets; gathered rows go straight from memory to
//               registers through buffer loads whose hardware range check
//               returns zero for absent neighbours; a 16-row block whose 16
//               rows all lack offset i skips its MFMAs (and, for filters
//               other than 3^3, its gathers).
//   k_fwd_lowc  at most 4 input planes (e.g. the 1 plane of a pen-stroke
//               input): one lane per (output row, 16 output columns), fp32
//               FMA chains, weights through the scalar cache.
//   k_fwd_slab  (forward_slab.h) any other channel count on the matrix cores,
//               rows walked in slabs of channels.
//   k_fwd_vec   layers that it finishes before k_fwd_slab (vec_first), or
//               operands past the buffer range: one lane per (output row,
//               output column), fp32 FMA chain.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "internal.h"

namespace spc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

// Test knob: SPCONV_FORCE_PATH=vec runs the vector path for shapes the
// matrix-core path would take; =slab runs k_fwd_slab for shapes that k_fwd_vec
// is estimated to finish first.
enum class Forced { kNone, kVec, kSlab };
Forced forced_path() {
  const char* e = std::getenv("SPCONV_FORCE_PATH");
  if (!e) return Forced::kNone;
  return std::strcmp(e, "vec") == 0    ? Forced::kVec
         : std::strcmp(e, "slab") == 0 ? Forced::kSlab
                                       : Forced::kNone;
}

constexpr uint32_t kBufDword3 = 0x00020000u;   // gfx9 raw buffer descriptor word 3

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// fp32 -> bf16, round to nearest even; NaN stays NaN.
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

template <typename T> struct ElemIO;
template <> struct ElemIO<float> {
  __device__ static float load(const float* p, int64_t i) { return p[i]; }
  __device__ static void store(float* p, int64_t i, float v) { p[i] = v; }
};
template <> struct ElemIO<uint16_t> {
  __device__ static float load(const uint16_t* p, int64_t i) { return bf16_to_f32(p[i]); }
  __device__ static void store(uint16_t* p, int64_t i, float v) { p[i] = f32_to_bf16(v); }
};

// Buffer loads whose hardware range check returns zero for an offset past
// the resource (kBufOOB and up): a load that may have nothing to read needs
// no branch (a load under a branch forces a wait for every load in flight).
constexpr uint32_t kBufOOB = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, static_cast<int>(bytes),
                                           static_cast<int>(kBufDword3));
}
template <typename T> struct BufIO;
template <> struct BufIO<float> {
  static constexpr uint32_t kSize = 4;
  __device__ static float load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
  }
};
template <> struct BufIO<uint16_t> {
  static constexpr uint32_t kSize = 2;
  __device__ static float load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    return bf16_to_f32(__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0));
  }
};
// Gather-map entries of offsets i0 .. i0 + KB - 1 at position p, minus one
// (-1: no neighbour, or offset past K).
template <int KB>
__device__ __forceinline__ void load_map(const int32_t* gmap, int64_t gstride, int K, int i0,
                                         int64_t p, int32_t (&g)[KB]) {
  const uint32_t bytes = static_cast<uint32_t>(gstride * 4);
#pragma unroll
  for (int b = 0; b < KB; ++b) {
    const int i = i0 + b < K ? i0 + b : 0;
    const __amdgpu_buffer_rsrc_t r = buf_rsrc(gmap + static_cast<int64_t>(i) * gstride, bytes);
    const uint32_t off = i0 + b < K ? static_cast<uint32_t>(p) * 4u : kBufOOB;
    g[b] = static_cast<int32_t>(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0)) - 1;
  }
}

// ---------------------------------------------------------------------------
// Generic (vector ALU) path
// ---------------------------------------------------------------------------
// Weight modes: the multiply-add uses Wk^i (C_in x C_out of the kernel) =
//   WT 0: w[i]                     (w is [K][C_in][C_out], the forward)
//   WT 2: w[i]^T                   (w is [K][C_out][C_in]: the input gradient of
//                                   SC / DC, run over the reversed pairs)
//   WT 1: w[K-1-i]^T               (the input gradient of VSC: its pairs are
//                                   symmetric, (a,b) in R_i iff (b,a) in R_{K-1-i})
template <int WT>
__device__ __forceinline__ int64_t w_index(int i, int K, int c, int n, int C_in, int C_out) {
  if constexpr (WT == 0) return (static_cast<int64_t>(i) * C_in + c) * C_out + n;
  const int iw = WT == 1 ? K - 1 - i : i;
  return (static_cast<int64_t>(iw) * C_out + n) * C_in + c;
}

// Epilogue and store of one output element (column col, element o of y).
template <typename TOut>
__device__ __forceinline__ void store_elem(float acc, int64_t o, int col, const float* bias,
                                           const Epilogue& epi, TOut* y) {
  if (epi.scale)
    acc = fmaf(acc, epi.scale[col], bias ? bias[col] : 0.0f);
  else if (bias)
    acc += bias[col];
  if (epi.res) acc += ElemIO<TOut>::load(static_cast<const TOut*>(epi.res), o);
  if (epi.relu) acc = acc < 0.0f ? 0.0f : acc;
  ElemIO<TOut>::store(y, o, acc);
}

// Positions run over the capacity n_cap (known on the host) so that the
// loads of the gather map do not wait for the device-side row count; a
// position at or past the count contributes nothing and stores nothing.
// The map entries of 8 offsets are loaded together (and, for one input
// plane, their input values and weights), then accumulated in offset order.
template <typename TIn, typename TOut, int WT>
__global__ __launch_bounds__(256) void k_fwd_vec(
    const int32_t* __restrict__ gmap, const int32_t* __restrict__ perm, int64_t gstride,
    int64_t n_cap, const DeviceHeader* __restrict__ hdr, int K, const TIn* __restrict__ x,
    const TIn* __restrict__ w, const float* __restrict__ bias, TOut* __restrict__ y, int C_in,
    int C_out, Epilogue epi) {
  constexpr int KB = 8;
  const int64_t n_rows = hdr->n_out;
  const int64_t total = n_cap * C_out;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; idx < total;
       idx += stride) {
    const int64_t p = idx / C_out;                 // schedule position
    const int col = static_cast<int>(idx - p * C_out);
    const bool live = p < n_rows;
    float acc = 0.0f;
    for (int i0 = 0; i0 < K; i0 += KB) {
      int32_t g[KB];
#pragma unroll
      for (int b = 0; b < KB; ++b) {          // in bounds for every b: no branch
        const int i = i0 + b < K ? i0 + b : K - 1;
        g[b] = gmap[static_cast<int64_t>(i) * gstride + p] - 1;
      }
#pragma unroll
      for (int b = 0; b < KB; ++b) g[b] = (live && i0 + b < K) ? g[b] : -1;
      if (C_in == 1) {
        float xv[KB], wv[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b) {
          xv[b] = g[b] >= 0 ? ElemIO<TIn>::load(x, g[b]) : 0.0f;
          wv[b] = i0 + b < K ? ElemIO<TIn>::load(w, w_index<WT>(i0 + b, K, 0, col, 1, C_out))
                             : 0.0f;
        }
#pragma unroll
        for (int b = 0; b < KB; ++b)
          if (g[b] >= 0) acc = fmaf(xv[b], wv[b], acc);
      } else {
#pragma unroll
        for (int b = 0; b < KB; ++b) {
          if (g[b] < 0) continue;
          const int64_t xb = static_cast<int64_t>(g[b]) * C_in;
          for (int c = 0; c < C_in; ++c)
            acc = fmaf(ElemIO<TIn>::load(x, xb + c),
                       ElemIO<TIn>::load(w, w_index<WT>(i0 + b, K, c, col, C_in, C_out)), acc);
        }
      }
    }
    if (live) store_elem(acc, static_cast<int64_t>(perm[p]) * C_out + col, col, bias, epi, y);
  }
}

// A pair view on the vector ALU, one lane per (pair, column).
template <typename TIn, typename TOut, int WT>
__global__ __launch_bounds__(256) void k_pairs_vec(
    const int32_t* __restrict__ pairs, const int64_t* __restrict__ pair_off, int K,
    const TIn* __restrict__ x, const TIn* __restrict__ w, const float* __restrict__ bias,
    TOut* __restrict__ y, int C_in, int C_out) {
  const int64_t total = pair_off[K] * C_out;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; t < total;
       t += stride) {
    const int64_t e = t / C_out;
    const int n = static_cast<int>(t % C_out);
    int i = 0, hi = K;                             // pair_off[i] <= e < pair_off[hi]
    while (hi - i > 1) {
      const int mid = (i + hi) / 2;
      if (pair_off[mid] <= e) i = mid; else hi = mid;
    }
    const int64_t xb = static_cast<int64_t>(pairs[2 * e + 1]) * C_in;
    float acc = 0.0f;
    for (int c = 0; c < C_in; ++c)
      acc = fmaf(ElemIO<TIn>::load(x, xb + c),
                 ElemIO<TIn>::load(w, w_index<WT>(i, K, c, n, C_in, C_out)), acc);
    store_elem(acc, static_cast<int64_t>(pairs[2 * e]) * C_out + n, n, bias, Epilogue{}, y);
  }
}

// Four adjacent output elements: rounded once and stored, or read as fp32 (the
// residual of the epilogue).
__device__ __forceinline__ void store4(float* p, const float* v) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void store4(uint16_t* p, const float* v) {
  uint2 u;
  u.x = f32_to_bf16(v[0]) | (static_cast<uint32_t>(f32_to_bf16(v[1])) << 16);
  u.y = f32_to_bf16(v[2]) | (static_cast<uint32_t>(f32_to_bf16(v[3])) << 16);
  *reinterpret_cast<uint2*>(p) = u;
}
__device__ __forceinline__ void load4(const float* p, float* v) {
  const float4 u = *reinterpret_cast<const float4*>(p);
  v[0] = u.x; v[1] = u.y; v[2] = u.z; v[3] = u.w;
}
__device__ __forceinline__ void load4(const uint16_t* p, float* v) {
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  v[0] = __uint_as_float(u.x << 16); v[1] = __uint_as_float(u.x & 0xffff0000u);
  v[2] = __uint_as_float(u.y << 16); v[3] = __uint_as_float(u.y & 0xffff0000u);
}

// Few input planes (C_in <= kLowCin, C_out a multiple of kLowCols): one
// thread per output position and kLowCols output columns, a block of threads
// on one column group.  The gather-map entries and input values of KB
// offsets at a time (9, or 16 for larger filters) are loaded together into
// registers; meanwhile the block stages those offsets' weights of its
// columns in LDS, which every lane then reads at the same address (a
// broadcast).  The finished rows go
// through LDS once more, so that each store instruction writes whole 16-byte
// pieces of few rows (4 lanes per row) instead of one element of 64 rows
// (on 476,000 pen-stroke rows, 1 -> 32 fp32: 40 us against 87 us; 32
// columns per thread instead of 16 took 106 us).  Same per-element summation
// order as k_fwd_vec.
constexpr int kLowCin = 4;
constexpr int kLowCols = 16;
template <typename TIn, typename TOut, int WT, int KB>
__global__ __launch_bounds__(256) void k_fwd_lowc(
    const int32_t* __restrict__ gmap, const int32_t* __restrict__ perm, int64_t gstride,
    int64_t n_cap, const DeviceHeader* __restrict__ hdr, int K, const TIn* __restrict__ x,
    const TIn* __restrict__ w, const float* __restrict__ bias, TOut* __restrict__ y, int C_in,
    int C_out, uint32_t x_bytes, Epilogue epi) {
  constexpr int NCOL = kLowCols;
  constexpr int kW = KB * kLowCin * NCOL;         // staged weights (floats)
  constexpr int kO = 4 * 64 * (NCOL + 1);         // finished rows, per wave 64 x NCOL (+1 pad)
  __shared__ float s_buf[kW > kO ? kW : kO];
  __shared__ int64_t s_row[256];
  float (*s_w)[kLowCin][NCOL] = reinterpret_cast<float (*)[kLowCin][NCOL]>(s_buf);
  const int64_t p = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  const int n0 = blockIdx.y * NCOL;               // first column of the block
  const __amdgpu_buffer_rsrc_t xr = buf_rsrc(x, x_bytes);
  const bool live = p < n_cap && p < hdr->n_out;
  const int64_t pc = p < n_cap ? p : 0;           // a position the map holds
  // the output row, loaded up front
  s_row[threadIdx.x] = live ? static_cast<int64_t>(perm[pc]) * C_out : -1;
  float acc[NCOL];
#pragma unroll
  for (int n = 0; n < NCOL; ++n) acc[n] = 0.0f;
  for (int i0 = 0; i0 < K; i0 += KB) {
    int32_t g[KB];
    load_map<KB>(gmap, gstride, K, i0, pc, g);
    float xv[KB][kLowCin];
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
      for (int c = 0; c < kLowCin; ++c) {
        xv[b][c] = 0.0f;
        if (c < C_in && i0 + b < K) {             // block-uniform
          const uint32_t off = (live && g[b] >= 0)
                                   ? (static_cast<uint32_t>(g[b]) * C_in + c) * BufIO<TIn>::kSize
                                   : kBufOOB;
          xv[b][c] = BufIO<TIn>::load(xr, off);
        }
      }
    if (i0 > 0) __syncthreads();                  // the last batch's weights are read
    for (int e = threadIdx.x; e < KB * kLowCin * NCOL; e += blockDim.x) {
      const int b = e / (kLowCin * NCOL), c = (e / NCOL) % kLowCin, n = e % NCOL;
      s_w[b][c][n] = (i0 + b < K && c < C_in)
                         ? ElemIO<TIn>::load(w, w_index<WT>(i0 + b, K, c, n0 + n, C_in, C_out))
                         : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      if (i0 + b < K) {
        const bool has = live && g[b] >= 0;
#pragma unroll
        for (int c = 0; c < kLowCin; ++c) {
          if (c < C_in) {
#pragma unroll
            for (int n = 0; n < NCOL; ++n)
              acc[n] = has ? fmaf(xv[b][c], s_w[b][c][n], acc[n]) : acc[n];
          }
        }
      }
    }
  }
  // rows -> LDS (the weights' space), then NCOL / 4 lanes per row store
  // 4 adjacent columns each
  __syncthreads();
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  float* s_o = s_buf + wave * 64 * (NCOL + 1);
#pragma unroll
  for (int n = 0; n < NCOL; ++n) s_o[lane * (NCOL + 1) + n] = acc[n];
  __syncthreads();
  constexpr int CG = NCOL / 4;                    // 4-column groups per row
#pragma unroll
  for (int k = 0; k < CG; ++k) {
    const int idx = k * 64 + lane;
    const int r = idx / CG, cg = idx % CG;
    const int64_t o = s_row[wave * 64 + r];
    if (o < 0) continue;
    const int col = n0 + cg * 4;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = s_o[r * (NCOL + 1) + cg * 4 + e];
      if (epi.scale)
        v[e] = fmaf(v[e], epi.scale[col + e], bias ? bias[col + e] : 0.0f);
      else if (bias)
        v[e] += bias[col + e];
    }
    if (epi.res) {
      float rv[4];
      load4(static_cast<const TOut*>(epi.res) + o + col, rv);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += rv[e];
    }
    if (epi.relu) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = v[e] < 0.0f ? 0.0f : v[e];
    }
    store4(y + o + col, v);
  }
}

// ---------------------------------------------------------------------------
// Matrix-core path
// ---------------------------------------------------------------------------
// Element traits: a lane moves 16 bytes per k-chunk; KC real k per chunk
// across the 4 lane groups of a 16x16 MFMA.
template <typename T> struct MT;
template <> struct MT<uint16_t> {          // bf16
  static constexpr int KC = 32;            // 8 bf16 per lane x 4 groups
  static constexpr int T = 8;              // transpose tile (elements per 16 B)
  __device__ static f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
template <> struct MT<float> {             // fp32
  static constexpr int KC = 16;            // 4 fp32 per lane x 4 groups
  static constexpr int T = 4;
  __device__ static f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
    // The 4 elements of a lane's 16-byte chunk are consumed by 4 MFMA steps;
    // step e pairs A[r][16ch + 4g + e] with B[16ch + 4g + e][c] in every lane
    // group g, so the 4 steps cover the chunk's 16 k exactly once.
#pragma unroll
    for (int e = 0; e < 4; ++e)
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(b[e]), c,
                                               0, 0, 0);
    return c;
  }
};

__device__ __forceinline__ u32x4 buf_load16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
}

// LDS image of W^i transposed: one row per output column of the chunk, ROWB
// bytes of k.  Rows whose length is a multiple of 128 bytes store 16-byte
// chunk c at c ^ swz(row), so that the fragment reads, where 8 lanes read one
// chunk of 8 consecutive rows, fall on different banks; a 16-byte pad per row,
// used for other lengths, leaves them a 2-way conflict.  The 4-byte writes of
// the staging come from lanes that hold every fourth row of one or of several
// blocks of 16 (TileCols): with row & 7 alone up to eight of them met on a bank.
// fp32: swz also takes the row's fourth bit and every block of 16 rows is
// shifted by half the banks (a quarter for a padded row) and a chunk, which
// costs the reads nothing: no two meet (16 -> 64 planes 5^2 3,305 pen rows 17.5
// -> 15.8 us, 29,760 rows 64 -> 64 3^3 32.3 -> 29.0).  128 bf16 planes: the bit
// alone, two meet (strided 3^3 of 345,353 rows, 128 -> 128: 163.6 -> 150.2 us).
// Fewer bf16 planes keep row & 7: 64 of them need their registers for a third
// workgroup (kNear), and 32 -> 64 5^2 lost 6 % by the shifts.
template <typename TIn, int ROWB>
struct WImage {
  static constexpr bool kSwz = ROWB % 128 == 0;
  static constexpr int kRowBytes = kSwz ? ROWB : ROWB + 16;
  __device__ static int swz(int row) {
    if constexpr (sizeof(TIn) == 4) return (row ^ (row >> 3 & 1) << 1) & 7;
    return ROWB < 256 ? row & 7 : (row ^ (row >> 3 & 1)) & 7;
  }
  __host__ __device__ static constexpr int shift(int block) {
    return sizeof(TIn) == 4 ? (kSwz ? 128 : 32) * block + 16 * (block >> 1) : 0;
  }
  static constexpr int bytes(int rows) { return rows * kRowBytes + shift(rows / 16 - 1); }
  __device__ static int at(int row, int byte) {
    const int base = row * kRowBytes + shift(row >> 4);
    if constexpr (kSwz)
      return base + ((((byte >> 4) ^ swz(row)) << 4) | (byte & 15));
    else
      return base + byte;
  }
};

// Gather-map entries of a wave's RB blocks of 16 rows, one load instruction
// per offset: lane l holds row l mod 16 RB of the wave (map_lane), and the
// matrix-core layout, where all four 16-lane groups need block b's 16 entries,
// comes from register swaps of 32- and 16-lane halves (spread_map).  One load
// per block instead kept three more registers per offset in flight (348,208
// surface rows 32 -> 32 fp32 3^3: 200 us against 186 us now; bf16 layers,
// which the gathers themselves bound, are the same within 1 %).
template <int RB>
__device__ __forceinline__ int map_lane(int lane) {
  return lane & (16 * RB - 1);
}
template <int RB>
__device__ __forceinline__ void spread_map(int32_t v, int32_t (&g)[RB]) {
  static_assert(RB == 1 || RB == 2 || RB == 4, "blocks of 16 rows in a wave of 64 lanes");
  const unsigned u = static_cast<unsigned>(v);
  if constexpr (RB == 1) {
    g[0] = v;
  } else if constexpr (RB == 2) {
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    g[0] = static_cast<int32_t>(a[0]);
    g[1] = static_cast<int32_t>(a[1]);
  } else {
    const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const auto a = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
    g[0] = static_cast<int32_t>(a[0]);
    g[1] = static_cast<int32_t>(a[1]);
    g[2] = static_cast<int32_t>(b[0]);
    g[3] = static_cast<int32_t>(b[1]);
  }
}
// The blocks (bit b) with at least one row present.
template <int RB>
__device__ __forceinline__ uint32_t map_blocks(int32_t v) {
  const uint64_t m = __ballot(v >= 0);
  uint32_t pres = 0;
#pragma unroll
  for (int b = 0; b < RB; ++b) pres |= ((m >> (16 * b)) & 0xffffu) != 0 ? 1u << b : 0u;
  return pres;
}

// 16 bytes of adjacent output elements, rounded once; and read back as fp32.
__device__ __forceinline__ void store16(float* p, const float* v) { store4(p, v); }
__device__ __forceinline__ void store16(uint16_t* p, const float* v) {
  uint4 u;
  u.x = f32_to_bf16(v[0]) | (static_cast<uint32_t>(f32_to_bf16(v[1])) << 16);
  u.y = f32_to_bf16(v[2]) | (static_cast<uint32_t>(f32_to_bf16(v[3])) << 16);
  u.z = f32_to_bf16(v[4]) | (static_cast<uint32_t>(f32_to_bf16(v[5])) << 16);
  u.w = f32_to_bf16(v[6]) | (static_cast<uint32_t>(f32_to_bf16(v[7])) << 16);
  *reinterpret_cast<uint4*>(p) = u;
}
template <typename TOut>
__device__ __forceinline__ float piece_elem(const u32x4& u, int e) {
  if constexpr (sizeof(TOut) == 4) return __uint_as_float(u[e]);
  return __uint_as_float(e & 1 ? u[e / 2] & 0xffff0000u : u[e / 2] << 16);
}

// Which columns a lane of a tile of NCB blocks ends with: W^T is the first
// operand of the products, so lane group g (lane / 16) holds, of row lane mod
// 16 of each row block, the results of LDS rows 16 cb + 4 g .. + 3 of every
// column block cb.  Runs of kRun adjacent columns are dealt to the four groups
// in turn: all 4 NCB of a lane's columns; 16 bytes of them for fp32, so that one
// store instruction writes 64 adjacent bytes of each of its 16 rows instead of
// 16 bytes in every 64 (348,208 rows 64 -> 64 of one offset 49.2 us, 43.1  now;
// bf16 stores 16 bytes in every 32 at most, and loses more registers than it
// gains; so do fp32 tiles of 32 columns on more offsets, whose stores are few:
// SHORT false, 29,760 pen rows 32 -> 32 3^2 11.2 us with short runs, 10.8 without).
template <typename TIn, typename TOut, int NCB, bool SHORT>
struct TileCols {
  static constexpr int kRun = SHORT && sizeof(TIn) == 4 && sizeof(TOut) == 4 ? 4 : 4 * NCB;
  // LDS row of column n
  __device__ static int row_of(int n) {
    if constexpr (kRun == 4 * NCB) return n % kRun / 4 * 16 + n / kRun * 4 + n % 4;
    const int q = n / (4 * kRun), g = n % (4 * kRun) / kRun, e = n % kRun;
    return 16 * (q * (kRun / 4) + e / 4) + 4 * g + e % 4;
  }
  // of a lane's 4 NCB columns, the e-th: where it lies past the first
  __device__ static constexpr int col(int e) { return e / kRun * 4 * kRun + e % kRun; }
};

// Epilogue of the matrix-core kernels: bias (scale, residual, ReLU), one
// rounding, the store, in 16-byte pieces (x as the first operand of the
// products leaves NCB columns of four rows per lane: 4- to 8-byte pieces and
// four times the row numbers; the 2^3 stride-2 layer 32 -> 64 of 1,703,204
// rows with its affine and ReLU fused took 102 us so, 78 us now; 902,504 rows
// 64 -> 64 3^3, with 207 registers instead of 225, 302 and 293 us).
// rowv: the output row of the wave's row map_lane (-1: none).  FULL: every
// column of the tile exists; otherwise columns past C_out are dropped, and rows
// that are no whole pieces go element by element.
template <typename TIn, typename TOut, int RB, int NCB, bool FULL, bool SHORT>
__device__ __forceinline__ void store_tile(const f32x4 (&acc)[RB][NCB], int32_t rowv,
                                           const float* bias, TOut* y, int C_out, int col0,
                                           int lg, const Epilogue& epi) {
  constexpr int LC = 4 * NCB;
  constexpr int P16 = 16 / static_cast<int>(sizeof(TOut));
  using TC = TileCols<TIn, TOut, NCB, SHORT>;
  constexpr int PC = LC < P16 ? LC : P16;         // (one block of bf16 columns: 8 bytes)
  constexpr int NP = LC / PC;
  const int n0 = col0 + lg * TC::kRun;            // the lane's e-th column: n0 + col(e)
  const bool whole = FULL || C_out % PC == 0;
  int32_t row[RB];
  spread_map<RB>(rowv, row);
  const TOut* res = static_cast<const TOut*>(epi.res);
  u32x4 rv[RB][NP];
  if (res && whole) {
    // all blocks' residual pieces first, so that their latencies overlap (a
    // row of -1 reads row 0, which exists whenever this tile runs)
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int n = n0 + TC::col(q * PC);
        const TOut* p = res + static_cast<int64_t>(row[b] >= 0 ? row[b] : 0) * C_out +
                        (FULL || n < C_out ? n : 0);
        if constexpr (PC == P16) {
          rv[b][q] = *reinterpret_cast<const u32x4*>(p);
        } else {
          const uint2 u = *reinterpret_cast<const uint2*>(p);
          rv[b][q] = u32x4{u.x, u.y, 0u, 0u};
        }
      }
  }
  float bv[LC], sv[LC];
#pragma unroll
  for (int e = 0; e < LC; ++e) {
    const int c = n0 + TC::col(e);
    const int n = FULL || c < C_out ? c : C_out - 1;
    bv[e] = bias ? bias[n] : 0.0f;
    sv[e] = epi.scale ? epi.scale[n] : 1.0f;
  }
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    if (row[b] < 0) continue;
    TOut* out = y + static_cast<int64_t>(row[b]) * C_out + n0;
    float z[LC];
#pragma unroll
    for (int e = 0; e < LC; ++e) {
      const float a = acc[b][e / 4][e % 4];
      z[e] = epi.scale ? fmaf(a, sv[e], bv[e]) : a + bv[e];
    }
    if (res) {
#pragma unroll
      for (int e = 0; e < LC; ++e) {
        if (whole)
          z[e] += piece_elem<TOut>(rv[b][e / PC], e % PC);
        else if (n0 + TC::col(e) < C_out)
          z[e] += ElemIO<TOut>::load(res, static_cast<int64_t>(row[b]) * C_out + n0 + TC::col(e));
      }
    }
    if (epi.relu) {
#pragma unroll
      for (int e = 0; e < LC; ++e) z[e] = z[e] < 0.0f ? 0.0f : z[e];
    }
    if (whole) {
#pragma unroll
      for (int q = 0; q < NP; ++q)
        if (FULL || n0 + TC::col(q * PC) < C_out) {
          if constexpr (PC == P16) store16(out + TC::col(q * PC), z + q * PC);
          else store4(out + TC::col(q * PC), z + q * PC);
        }
    } else {
#pragma unroll
      for (int e = 0; e < LC; ++e)
        if (n0 + TC::col(e) < C_out)
          ElemIO<TOut>::store(out, TC::col(e), z[e]);
    }
  }
}

// Pair views: the tiles of offset i are runs of ROWS of its pairs.  They sit in
// the slots from pair_off[i] / ROWS + i on (both rounded down), which are at
// least as many as the offset's tiles, so no list or sum of tile counts is
// needed to find a slot's offset: the last one whose first slot is not past
// it.  At most one slot per offset holds no pairs; the XCDs get contiguous
// ranges of slots.
struct PairTile {
  int i, count;                // offset; pairs (fewer than ROWS at the end of R_i)
  int64_t first;               // first pair
};
template <int ROWS>
__device__ __forceinline__ bool pair_tile(const int64_t* __restrict__ pair_off, int K,
                                          int64_t nslots, PairTile* t) {
  const int64_t per = (nslots + 7) / 8, q8 = blockIdx.x / 8;
  const int64_t slot = static_cast<int64_t>(blockIdx.x % 8) * per + q8;
  if (q8 >= per || slot >= nslots) return false;
  // the wave looks at every J-th offset, then (J > 1) at those in between
  static_assert(kMaxK <= kWave * kWave, "two looks");
  const int lane = __lane_id(), J = (K + kWave - 1) / kWave;
  auto last = [&](int i, bool in) -> int {         // the last lane whose offset starts in time
    const int64_t off = pair_off[in ? i : K];
    return 63 - __builtin_clzll(__ballot(in && off / ROWS + i <= slot) | 1ull);
  };
  int i = J * last(J * lane, J * lane < K);
  if (J > 1) i += last(i + lane, lane < J && i + lane < K);
  const int64_t lo = pair_off[i], k = pair_off[i + 1] - lo;
  const int64_t e = (slot - lo / ROWS - i) * ROWS;
  if (e >= k) return false;
  t->i = i;
  t->first = lo + e;
  t->count = static_cast<int>(k - e < ROWS ? k - e : ROWS);
  return true;
}
// The input row (which 0) or output row (1) of pair e of the tile, -1 past its
// end; a buffer load without a branch, as the map's.
__device__ __forceinline__ int32_t pair_row(const int32_t* pairs, const PairTile& t, int e,
                                            int which) {
  const __amdgpu_buffer_rsrc_t r =
      buf_rsrc(pairs + 2 * t.first, static_cast<uint32_t>(t.count) * 8u);
  const int32_t v = static_cast<int32_t>(
      __builtin_amdgcn_raw_buffer_load_b32(r, static_cast<uint32_t>(8 * e + 4 * which), 0, 0));
  return e < t.count ? v : -1;
}
// The arguments of a kernel on a view: a pair view's pairs, offsets and pair_K
// stand in for the map, the schedule and K.
struct ViewArgs {
  const int32_t* gmap;
  const int32_t* perm;
  int K;
};
inline ViewArgs view_args(const FwdView& v) {
  if (v.pair_off) return {v.pairs, reinterpret_cast<const int32_t*>(v.pair_off), v.pair_K};
  return {v.gmap, v.perm, static_cast<int>(v.K)};
}
// Tiles (slots, for pair views) of a launch on a view.
inline int64_t view_tiles(const FwdView& v, int rows) {
  return v.pair_off ? v.n_cap / rows + v.pair_K : (v.n_cap + rows - 1) / rows;
}

// -1 as a value the compiler does not know.  The offset whose W is staged is
// chosen against it at every step: left to itself the compiler carries a 64-bit
// address per staged piece through the offset loop (128 -> 128 bf16 with RB = 1:
// 173 registers instead of 153, two workgroups per compute unit instead of
// three).
__device__ __forceinline__ int unknown_minus_one() {
  int v;
  asm("s_mov_b32 %0, -1" : "=s"(v));
  return v;
}

// Tile of the output handled by one workgroup: 4 waves x RB blocks of 16 rows,
// NCB blocks of 16 columns (the whole workgroup shares one column chunk).
//
// Lane layout (16x16 MFMA): lane l = 16 g + r.  Gathered rows (second operand):
// row r of the 16-row block, k-chunk bytes [16 g, 16 g + 16).  W^T (first
// operand): LDS row 16 cb + r of the chunk, same k bytes.  Result: lane l holds
// row r's products with LDS rows 16 cb + 4 g + v (v = 0..3), whose columns
// TileCols says.
//
// Pipeline over the offsets (iteration i): G(i+3) and W^(i+2) are fetched,
// gathered rows A(i+2) are issued (their gather-map entries G(i+2) arrived
// one iteration earlier), the MFMAs of offset i run on A(i) and the LDS copy
// of W^i, and W^(i+1) (fetched one iteration earlier) is written transposed
// into the other LDS buffer.  One barrier per offset publishes W^(i+1).
//
// kNear (64 bf16 planes to 64 columns per tile, 27 offsets): rows and W^i are
// requested one offset ahead instead of two, into two row sets instead of
// three; 167 registers instead of 207 let three workgroups share a compute
// unit instead of two, which hides more than the longer distance does
// (902,504 surface rows 64 -> 64 3^3: 298 -> 284 us).  Other shapes gain no
// workgroup by it, or lose (128 planes: 53 -> 68 us, RB = 2; 32 planes, which
// go from four to five, are the same).
template <typename TIn, int NCH, int NCB, int RB, int KT>
constexpr bool kNear = sizeof(TIn) == 2 && NCH == 2 && NCB == 4 && RB == 4 && KT == 27;
template <typename TIn, int NCH, int NCB, int RB, typename TOut, int KT, bool SKIP = false,
          int WT = 0, bool LSKIP = false, bool PAIRS = false>
__global__ __launch_bounds__(256, (kNear<TIn, NCH, NCB, RB, KT> ? 3 : 2)) void k_fwd_mfma(
    const int32_t* __restrict__ gmap, const int32_t* __restrict__ perm, int64_t gstride,
    const DeviceHeader* __restrict__ hdr, int K_arg,
    const TIn* __restrict__ x, uint32_t x_bytes, const TIn* __restrict__ w,
    const float* __restrict__ bias, TOut* __restrict__ y, int C_out, int64_t ntiles,
    Epilogue epi) {
  // KT > 0: the offset count is a compile-time constant and the offset loop
  // is unrolled completely (no loop-carried register hazards).
  // PAIRS (KT = 1): a pair view, from which the tile's rows and its W^i come;
  // its pairs, their offsets and its K are in the map's, the schedule's and K's
  // arguments (longer argument lists cost every launch: 16 bytes 0.2 us).
  static_assert(!PAIRS || KT == 1, "a pair view has one offset per tile");
  const int K = KT > 0 ? KT : K_arg;
  constexpr int KC = MT<TIn>::KC;
  constexpr int CIN = NCH * KC;
  constexpr int COLS = NCB * 16;
  constexpr int ESZ = static_cast<int>(sizeof(TIn));
  constexpr int ROWB = CIN * ESZ;                 // bytes of one input row
  // W^T staging tasks: bf16 takes 2 k-rows x 8 columns (packed in pairs),
  // fp32 1 k-row x 4 columns; each task is one 16-byte load per k-row.
  constexpr int KPT = ESZ == 2 ? 2 : 1;           // k-rows per task
  constexpr int NPT = 16 / ESZ;                   // columns per task
  constexpr int NTASK = (CIN / KPT) * (COLS / NPT);
  constexpr int TPT = (NTASK + 255) / 256;        // tasks per thread
  constexpr int WAVE_ROWS = RB * 16;
  constexpr int TILE_ROWS = 4 * WAVE_ROWS;

  __shared__ __attribute__((aligned(16))) unsigned char s_w[2][WImage<TIn, ROWB>::bytes(COLS)];

  // XCD-aware tile order: workgroup b runs on XCD b % 8; give each XCD a
  // contiguous range of tiles so neighbouring tiles share that XCD's L2.  The
  // grid is sized for a bound on the rows (an SC output count is known only
  // on the device), so the ranges split the device-side tile count, not the
  // grid: otherwise a loose bound would leave whole XCDs without work.
  PairTile pt{0, 0, 0};
  int64_t n_rows = TILE_ROWS, tile = 0;
  if constexpr (PAIRS) {
    if (!pair_tile<TILE_ROWS>(reinterpret_cast<const int64_t*>(perm), K_arg, ntiles, &pt)) return;
  } else {
    n_rows = hdr->n_out;
    const int64_t nt_real = (n_rows + TILE_ROWS - 1) / TILE_ROWS;
    const int64_t nt = nt_real < ntiles ? nt_real : ntiles;
    const int64_t per = (nt + 7) / 8;
    const int64_t q = blockIdx.x / 8;
    if (q >= per) return;
    tile = static_cast<int64_t>(blockIdx.x % 8) * per + q;
    if (tile >= nt) return;
  }

  const int fixed = PAIRS ? pt.i : unknown_minus_one();   // the tile's only W^i, or -1

  const int col0 = blockIdx.y * COLS;
  const int wave = threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  const int lr = lane % 16, lg = lane / 16;
  const int64_t row0 = tile * TILE_ROWS + wave * WAVE_ROWS;

  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<TIn*>(x), 0, static_cast<int>(x_bytes),
                                        static_cast<int>(kBufDword3));
  constexpr uint32_t kOOB = 0x80000000u;   // past any x_bytes < 2^31: reads as zero

  // ---- W^i -> registers.  WT 0: task t = (k-row group kt, column group nt)
  // with nt fastest, so consecutive lanes read one k-row of the chunk end to
  // end.  WT 1/2: w holds W^T, one memory row per output column n with all k
  // contiguous; task t = (column n, 16-byte chunk kc of that row), kc fastest.
  constexpr int NGRP = COLS / NPT;                // column groups per k-row
  constexpr int CPR = ROWB / 16;                  // 16-byte chunks per W^T row
  constexpr int NTASK_T = COLS * CPR;
  constexpr int TPT_T = (NTASK_T + 255) / 256;
  constexpr int NWR = WT == 0 ? TPT * KPT : TPT_T;
  typedef u32x4 WRegs[NWR];
  auto w_load = [&](int i, WRegs& wr) {
    if (i >= K) return;
    if constexpr (WT == 0) {
#pragma unroll
      for (int q = 0; q < TPT; ++q) {
        // tasks beyond NTASK (only when NTASK is not a multiple of 256) re-read
        // task 0 and are never stored
        const int t0 = threadIdx.x + q * 256;
        const int t = (NTASK % 256 == 0 || t0 < NTASK) ? t0 : 0;
        const int kt = t / NGRP, nt = t % NGRP;
        const int iv = fixed >= 0 ? fixed : i;
        const TIn* src = w + (static_cast<int64_t>(iv) * CIN + kt * KPT) * C_out + col0 + nt * NPT;
#pragma unroll
        for (int r = 0; r < KPT; ++r)
          wr[q * KPT + r] = *reinterpret_cast<const u32x4*>(src + static_cast<int64_t>(r) * C_out);
      }
    } else {
      const int iw = fixed >= 0 ? fixed : (WT == 1 ? K - 1 - i : i);
#pragma unroll
      for (int q = 0; q < TPT_T; ++q) {
        const int t0 = threadIdx.x + q * 256;
        const int t = (NTASK_T % 256 == 0 || t0 < NTASK_T) ? t0 : 0;
        const int n = t / CPR, kc = t % CPR;
        const TIn* src = w + (static_cast<int64_t>(iw) * C_out + col0 + n) * CIN + kc * (16 / ESZ);
        wr[q] = *reinterpret_cast<const u32x4*>(src);
      }
    }
  };
  // ---- registers -> LDS, transposed: one LDS row per column n holding
  // W^i[k][n] for all k (TileCols); the lanes that read one fragment chunk
  // together read 16 consecutive rows (spread over the banks by WImage).
  constexpr bool kShort = NCB >= 4 || KT == 1;
  auto w_row = [](int n) { return TileCols<TIn, TOut, NCB, kShort>::row_of(n); };
  auto w_store = [&](int i, const WRegs& wr) {
    if (i >= K) return;
    unsigned char* dst = s_w[i & 1];
    if constexpr (WT == 0) {
#pragma unroll
      for (int q = 0; q < TPT; ++q) {
        const int t = threadIdx.x + q * 256;
        if (NTASK % 256 == 0 || t < NTASK) {
          const int kt = t / NGRP, nt = t % NGRP;
          if constexpr (ESZ == 2) {
            // pack (W[2kt][n], W[2kt+1][n]) into one 32-bit LDS word per column
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const uint32_t a = wr[q * KPT][j / 2], b = wr[q * KPT + 1][j / 2];
              const uint32_t v = (j & 1) ? ((a >> 16) | (b & 0xffff0000u))
                                         : ((a & 0xffffu) | (b << 16));
              *reinterpret_cast<uint32_t*>(&dst[WImage<TIn, ROWB>::at(w_row(nt * 8 + j), kt * 4)]) = v;
            }
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              *reinterpret_cast<uint32_t*>(&dst[WImage<TIn, ROWB>::at(w_row(nt * 4 + j), kt * 4)]) =
                  wr[q][j];
          }
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < TPT_T; ++q) {
        const int t = threadIdx.x + q * 256;
        if (NTASK_T % 256 == 0 || t < NTASK_T) {
          const int n = t / CPR, kc = t % CPR;
          *reinterpret_cast<u32x4*>(&dst[WImage<TIn, ROWB>::at(w_row(n), kc * 16)]) = wr[q];
        }
      }
    }
  };

  // ---- gather-map entries of this wave's rows (1 + input row, 0 = none)
  // through buffer loads: an offset past the map's range reads 0, so rows past
  // the end and offsets past K need no branch (a load under a divergent branch
  // would force a full wait for every load in flight).
  typedef int32_t GRegs;
  const uint32_t gmap_bytes = static_cast<uint32_t>(gstride * 4);
  const int64_t map_row = row0 + map_lane<RB>(lane);
  const uint32_t map_off = map_row < n_rows ? static_cast<uint32_t>(map_row) * 4u : kOOB;
  auto g_load = [&](int i, GRegs& g) {
    if constexpr (PAIRS) {
      g = i < K ? pair_row(gmap, pt, static_cast<int>(map_row), 1) : -1;
      return;
    }
    const int ic = i < K ? i : 0;
    const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int32_t*>(gmap + static_cast<int64_t>(ic) * gstride), 0,
        static_cast<int>(gmap_bytes), static_cast<int>(kBufDword3));
    g = static_cast<int32_t>(
            __builtin_amdgcn_raw_buffer_load_b32(gr, i < K ? map_off : kOOB, 0, 0)) - 1;
  };
  // ---- gathered rows; returns the blocks (bit b) with at least one row
  typedef u32x4 ARegs[RB][NCH];
  auto a_load = [&](const GRegs& gv, ARegs& a) -> uint32_t {
    const uint32_t pres = map_blocks<RB>(gv);
    int32_t g[RB];
    spread_map<RB>(gv, g);
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const uint32_t base = g[b] >= 0 ? static_cast<uint32_t>(g[b]) * ROWB + lg * 16 : kOOB;
      if (!LSKIP || (pres & (1u << b))) {
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch)
          a[b][ch] = buf_load16(xr, base == kOOB ? kOOB : base + ch * 64);
      } else {
        // a block with no row at this offset: no loads (its products are
        // skipped as well)
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) a[b][ch] = u32x4{0u, 0u, 0u, 0u};
      }
    }
    return pres;
  };

  f32x4 acc[RB][NCB];
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[b][cb] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto mma = [&](int i, const ARegs& a, uint32_t pres) {
    const unsigned char* sw = s_w[i & 1];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      u32x4 bw[NCB];                               // W^i fragments of chunk ch
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
        bw[cb] = *reinterpret_cast<const u32x4*>(
            &sw[WImage<TIn, ROWB>::at(cb * 16 + lr, ch * 64 + lg * 16)]);
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        if (SKIP && !(pres & (1u << b))) continue;   // all 16 rows lack offset i
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          acc[b][cb] = MT<TIn>::mma(bw[cb], a[b][ch], acc[b][cb]);
      }
    }
  };

  if constexpr (kNear<TIn, NCH, NCB, RB, KT>) {
    // two row sets: iteration i multiplies A(i) while A(i+1) and W^(i+1) come;
    // G(i+2) is requested before them, for the in-order load counter
    GRegs g0, g1;
    ARegs a0, a1;
    WRegs w0;
    uint32_t p0 = 0, p1 = 0;
    g_load(0, g0);
    g_load(1, g1);
    w_load(0, w0);
    p0 = a_load(g0, a0);
    w_store(0, w0);
    __syncthreads();
    auto step = [&](int i, ARegs& aU, uint32_t& pU, ARegs& aF, uint32_t& pF, GRegs& gU,
                    GRegs& gF) {
      if (i >= K) return;
      g_load(i + 2, gU);
      w_load(i + 1, w0);
      pF = a_load(gF, aF);
      mma(i, aU, pU);
      w_store(i + 1, w0);
      __syncthreads();
    };
#pragma unroll
    for (int i = 0; i < KT; i += 2) {
      step(i, a0, p0, a1, p1, g0, g1);
      step(i + 1, a1, p1, a0, p0, g1, g0);
    }
  } else {
    // Three rotating register sets (offsets i, i+1, i+2 modulo 3).
    GRegs g0, g1, g2;
    ARegs a0, a1, a2;
    WRegs w0, w1, w2;
    uint32_t p0 = 0, p1 = 0, p2 = 0;

    // prologue: W^0 into LDS, W^1 in registers, A(0), A(1), G(2) in flight
    g_load(0, g0);
    g_load(1, g1);
    g_load(2, g2);
    w_load(0, w0);
    w_load(1, w1);
    p0 = a_load(g0, a0);
    p1 = a_load(g1, a1);
    w_store(0, w0);
    __syncthreads();

    // iteration i uses set (i mod 3): A(i) in aU, G(i+2) in gF -> A(i+2) into aF,
    // G(i+3) into gU; W^(i+1) stored from wN, W^(i+2) loaded into wF.
    auto step = [&](int i, ARegs& aU, uint32_t& pU, ARegs& aF, uint32_t& pF, GRegs& gU,
                    GRegs& gF, WRegs& wN, WRegs& wF) {
      if (i >= K) return;
      // issue order matters: the in-order load counter lets a later wait for
      // G(i+3) or W^(i+2) leave the gathered rows issued after them in flight
      g_load(i + 3, gU);
      w_load(i + 2, wF);
      pF = a_load(gF, aF);
      mma(i, aU, pU);
      w_store(i + 1, wN);
      __syncthreads();
    };
    if constexpr (KT > 0) {
#pragma unroll
      for (int i = 0; i < KT; i += 3) {
        step(i, a0, p0, a2, p2, g0, g2, w1, w2);
        step(i + 1, a1, p1, a0, p0, g1, g0, w2, w0);
        step(i + 2, a2, p2, a1, p1, g2, g1, w0, w1);
      }
    } else {
      for (int i = 0; i < K; i += 3) {
        step(i, a0, p0, a2, p2, g0, g2, w1, w2);
        step(i + 1, a1, p1, a0, p0, g1, g0, w2, w0);
        step(i + 2, a2, p2, a1, p1, g2, g1, w0, w1);
      }
    }
  }

  int32_t row = -1;
  if constexpr (PAIRS) row = pair_row(gmap, pt, static_cast<int>(map_row), 0);
  else if (map_row < n_rows) row = perm[map_row];
  store_tile<TIn, TOut, RB, NCB, true, kShort>(acc, row, bias, y, C_out, col0, lg, epi);
}

// ---------------------------------------------------------------------------
// Dispatch
// ---------------------------------------------------------------------------
// Row blocks per wave: fewer when the input rows are wide, so that the two
// register sets of gathered rows (current and next offset) still fit.
template <int NCH>
constexpr int rows_blocks() { return NCH <= 2 ? 4 : (NCH <= 4 ? 2 : 1); }

using Call = FwdCall;

// Tiles of fewer rows (one 16-row block per wave) when a layer is too small
// to give every compute unit two tiles of the usual size: a 64-row tile per
// workgroup keeps all of them busy on small layers (filters other than the
// unrolled 3^3 / 2^3 / 1^d ones).
constexpr int64_t kSmallLayerTiles = 512;

template <typename TIn, int NCH, int NCB, typename TOut, int WT, int RB, bool SMALL = false>
void launch_mfma_rb(const Call& c) {
  constexpr int kTileRows = 4 * RB * 16;
  const int64_t ntiles = view_tiles(c.v, kTileRows);
  const int64_t per = (ntiles + 7) / 8;
  dim3 grid(static_cast<unsigned>(8 * per), static_cast<unsigned>(c.C_out / (NCB * 16)));
  // Whole 16-row blocks that lack an offset skip their products.  3^3
  // filters run the unrolled kernel; other filters (strided SC, DC and the
  // SC input gradient, whose rows come ordered by offset class so that most
  // blocks take one offset only) also skip the blocks' gathers.
  // Single-offset views (the pairs of f = s books, 1^d filters) unroll to one
  // step with a third of the registers, so more workgroups share a CU.
  auto kern = k_fwd_mfma<TIn, NCH, NCB, RB, TOut, 0, true, WT, true>;
  if constexpr (!SMALL) {
    kern = c.v.K == 27  ? k_fwd_mfma<TIn, NCH, NCB, RB, TOut, 27, true, WT>
           : c.v.K == 1 ? k_fwd_mfma<TIn, NCH, NCB, RB, TOut, 1, true, WT>
           : c.v.K == 8 ? k_fwd_mfma<TIn, NCH, NCB, RB, TOut, 8, true, WT, true>
                        : kern;
    if constexpr (WT != 1)
      if (c.v.pair_off) kern = k_fwd_mfma<TIn, NCH, NCB, RB, TOut, 1, true, WT, false, true>;
  }
  const ViewArgs a = view_args(c.v);
  kern<<<grid, 256, 0, c.stream>>>(
      a.gmap, a.perm, c.v.gstride, c.v.hdr, a.K, static_cast<const TIn*>(c.x), c.x_bytes,
      static_cast<const TIn*>(c.w), c.bias, static_cast<TOut*>(c.y), c.C_out, ntiles, c.epi);
}

template <typename TIn, int NCH, int NCB, typename TOut, int WT>
void launch_mfma(const Call& c) {
  constexpr int RB = rows_blocks<NCH>();
  const bool generic_k = c.v.K != 27 && c.v.K != 1 && c.v.K != 8;
  const int64_t tiles = (c.v.n_cap + 4 * RB * 16 - 1) / (4 * RB * 16);
  if constexpr (RB > 1) {
    if (generic_k && tiles < kSmallLayerTiles) {
      launch_mfma_rb<TIn, NCH, NCB, TOut, WT, 1, true>(c);
      return;
    }
  }
  launch_mfma_rb<TIn, NCH, NCB, TOut, WT, RB>(c);
}

template <typename TIn, int NCH, typename TOut, int WT>
void launch_mfma_ncb(const Call& c) {
  // wide fp32 rows leave no registers for 4 column blocks
  constexpr bool four = !(sizeof(TIn) == 4 && NCH >= 6);
  if (four && c.C_out % 64 == 0)
    launch_mfma<TIn, NCH, four ? 4 : 2, TOut, WT>(c);
  else if (c.C_out % 32 == 0)
    launch_mfma<TIn, NCH, 2, TOut, WT>(c);
  else
    launch_mfma<TIn, NCH, 1, TOut, WT>(c);
}

template <typename TOut, int WT>
bool try_mfma(const Call& c, int in_dt, int C_in) {
  if (c.C_out % 16 != 0) return false;
  const uint64_t xb = static_cast<uint64_t>(c.v.n_src) * C_in * (in_dt == SPCONV_BF16 ? 2 : 4);
  // buffer ranges are kept below 2^31 bytes (inputs and one offset's map row)
  if (xb >= 0x7fffffffull || static_cast<uint64_t>(c.v.gstride) * 4 >= 0x7fffffffull) return false;
  Call cc = c;
  cc.x_bytes = static_cast<uint32_t>(xb);
  if (in_dt == SPCONV_BF16) {
    switch (C_in) {
      case 32: launch_mfma_ncb<uint16_t, 1, TOut, WT>(cc); return true;
      case 64: launch_mfma_ncb<uint16_t, 2, TOut, WT>(cc); return true;
      case 96: launch_mfma_ncb<uint16_t, 3, TOut, WT>(cc); return true;
      case 128: launch_mfma_ncb<uint16_t, 4, TOut, WT>(cc); return true;
      default: return false;
    }
  }
  switch (C_in) {
    case 16: launch_mfma_ncb<float, 1, TOut, WT>(cc); return true;
    case 32: launch_mfma_ncb<float, 2, TOut, WT>(cc); return true;
    case 64: launch_mfma_ncb<float, 4, TOut, WT>(cc); return true;
    case 96: launch_mfma_ncb<float, 6, TOut, WT>(cc); return true;
    case 128: launch_mfma_ncb<float, 8, TOut, WT>(cc); return true;
    default: return false;
  }
}

template <typename TIn, typename TOut, int WT>
void launch_vec(const Call& c, int C_in) {
  const int64_t total = c.v.n_cap * c.C_out;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  if (c.v.pair_off) {
    k_pairs_vec<TIn, TOut, WT><<<static_cast<unsigned>(blocks), 256, 0, c.stream>>>(
        c.v.pairs, c.v.pair_off, c.v.pair_K, static_cast<const TIn*>(c.x),
        static_cast<const TIn*>(c.w), c.bias, static_cast<TOut*>(c.y), C_in, c.C_out);
    return;
  }
  k_fwd_vec<TIn, TOut, WT><<<static_cast<unsigned>(blocks), 256, 0, c.stream>>>(
      c.v.gmap, c.v.perm, c.v.gstride, c.v.n_cap, c.v.hdr, static_cast<int>(c.v.K),
      static_cast<const TIn*>(c.x), static_cast<const TIn*>(c.w), c.bias, static_cast<TOut*>(c.y),
      C_in, c.C_out, c.epi);
}

template <typename TIn, typename TOut, int WT>
void launch_lowc(const Call& c, int C_in, uint32_t x_bytes) {
  const dim3 grid(static_cast<unsigned>((c.v.n_cap + 255) / 256),
                  static_cast<unsigned>(c.C_out / kLowCols));
  // offsets in batches of KB: 9 covers a 3x3 filter in one batch (no map
  // loads for offsets past K), 16 anything larger
  auto kern = c.v.K <= 9 ? k_fwd_lowc<TIn, TOut, WT, 9> : k_fwd_lowc<TIn, TOut, WT, 16>;
  kern<<<grid, 256, 0, c.stream>>>(
      c.v.gmap, c.v.perm, c.v.gstride, c.v.n_cap, c.v.hdr, static_cast<int>(c.v.K),
      static_cast<const TIn*>(c.x), static_cast<const TIn*>(c.w), c.bias, static_cast<TOut*>(c.y),
      C_in, c.C_out, x_bytes, c.epi);
}

// Columns of a launch whose column tiles (64 at least where there are this
// many) are the grid's second dimension.
constexpr int kMaxTileCols = 65535 * 64;

template <typename TIn, typename TOut>
constexpr auto slab_entry() {
  if constexpr (sizeof(TIn) == 4) return sizeof(TOut) == 4 ? forward_slab_ff : forward_slab_fb;
  else return sizeof(TOut) == 4 ? forward_slab_bf : forward_slab_bb;
}

// Which of k_fwd_vec and k_fwd_slab finishes a layer first, by what each one's
// time goes with (us; one set of constants for all sizes, fitted to both kernels
// on 3,996 layers: 400 to 345,353 rows, 9 to 27 offsets, 1 to 96 planes to 1 to
// 128, both types: the kernel taken is at most 10 % slower than the other in
// 98 % of them).
//   k_fwd_vec   a serial chain of K' C_in multiply-adds per column, or, where
//               the lanes fill the device, rows x C_out x (K' C_in + 2 K), and
//               twice that for inputs past an XCD's 4 MB of L2; as for up to
//               four columns where fewer share a row's loads.  K': the offsets
//               that one row can have, all K but in the reversed direction of a
//               strided layer (3^3 stride 2: 8 of 27).
//   k_fwd_slab  K steps per k-chunk of channels: a step's latency where the
//               tiles fit the device at once, else rows x column tiles; up to
//               double for rows of x or W that are no whole 16-byte pieces, more
//               with the columns per tile where both are, and less in the
//               reversed direction, whose rows come ordered by their offsets.
// Measured (vec / slab us): few rows make the chain the shorter one (400 rows,
// 25 offsets, fp32 8 -> 128: 15 / 34; bf16 5 -> 10: 12 / 25; 21,774 surface
// rows 3^3 bf16 3 -> 10: 14 / 31), as do few columns of few planes (400,000
// rows fp32 1 -> 8: 68 / 200) and few offsets (345,353 rows bf16 12 -> 4
// reversed: 48 / 174); whole pieces or more columns the matrix cores (345,353
// rows fp32 16 -> 4: 255 / 97, 8 -> 16: 421 / 97; 400 rows, 9 offsets 32 -> 24:
// 27 / 8).
template <typename TIn>
inline bool vec_first(const FwdView& v, int C_in, int C_out, bool w_rows_whole) {
  constexpr bool f32 = sizeof(TIn) == 4;
  constexpr int P = 16 / static_cast<int>(sizeof(TIn));
  // (n_cap is a loose bound on the rows of an SC book whose filter exceeds its
  // stride, see launch_slab_cols; the vector kernel's grid covers all of it)
  const double n = static_cast<double>(v.n_src > 0 ? std::min(v.n_src, v.n_cap) : v.n_cap);
  const double k = static_cast<double>(v.K), kr = static_cast<double>(v.K_row);
  const bool some = v.K_row < v.K, ax = C_in % P == 0, aw = w_rows_whole;
  const double chain = std::max(5.0, (some ? 0.1 : 0.085) * kr * C_in);
  // (of the reversed direction's source rows, far fewer than n, less is read again)
  const bool past_l2 = n * C_in * sizeof(TIn) > ((some ? 24 : 4) << 20);
  const double lanes = (past_l2 ? 5.5e-7 : 2.7e-7) * static_cast<double>(v.n_cap) *
                       std::max<double>(C_out, std::min(4.0, C_in / 6.0)) *
                       (kr * C_in + 2.0 * k);
  double latency, rate;                    // us per step; us per step, row and column tile
  int col_tiles = (C_out + 63) / 64;
  if (ax && aw) {
    const int cb = (C_out + 15) / 16, chunks = (cb + 7) / 8, ncb = (cb + chunks - 1) / chunks;
    const double wide = ncb <= 2 ? 1.0 : ncb <= 4 ? (f32 ? 1.3 : 1.1) : (f32 ? 3.5 : 2.0);
    latency = (f32 ? 0.56 : 0.35) * wide * (some ? 0.4 : 1.0);
    rate = (f32 ? 9.6e-6 : 6.3e-6) * wide * (some ? 0.75 : 1.0);
    col_tiles = chunks;
  } else if (f32) {
    latency = some ? 0.6 : 0.77;
    rate = ax ? 1.85e-5 : 2.1e-5;
  } else {
    latency = aw ? 0.62 : ax ? 0.84 : 0.9;
    rate = aw ? 1.0e-5 * (1.0 + 0.04 * C_in) : ax ? 1.35e-5 : 1.45e-5 * (1.0 + 0.025 * C_in);
  }
  const double steps = k * ((C_in + MT<TIn>::KC - 1) / MT<TIn>::KC);
  return 3.0 + std::hypot(chain, lanes) <= 4.2 + steps * std::max(latency, rate * n * col_tiles);
}

// Channel counts k_fwd_mfma is not compiled for.
template <typename TIn, typename TOut, int WT>
void launch_generic(const Call& c, int C_in, Forced forced) {
  // buffer ranges (inputs, weights, one offset's map row) are kept below 2^31
  // bytes; lowc also needs one grid row of blocks per kLowCols columns (at
  // most 65535).  Below kLowMinRows positions of few planes the
  // one-lane-per-column kernel finishes first (measured: 460 rows of 16
  // columns 6.1 us against 7.7 us; 29759 rows of 32 columns 16.4 us against
  // 12.7 us).
  constexpr int64_t kLowMinRows = 2048;
  const uint64_t xb = static_cast<uint64_t>(c.v.n_src) * C_in * sizeof(TIn);
  const bool by_pairs = c.v.pair_off != nullptr;
  const uint64_t wb =
      static_cast<uint64_t>(by_pairs ? c.v.pair_K : c.v.K) * C_in * c.C_out * sizeof(TIn);
  const bool fits = xb < kBufOOB && static_cast<uint64_t>(c.v.gstride) * 4 < kBufOOB;
  if (!by_pairs && C_in <= kLowCin && fits && c.v.n_cap >= kLowMinRows &&
      c.C_out % kLowCols == 0 && c.C_out / kLowCols <= 65535) {
    launch_lowc<TIn, TOut, WT>(c, C_in, static_cast<uint32_t>(xb));
    return;
  }
  const bool wfits = wb < kBufOOB && c.C_out <= kMaxTileCols;
  const bool w_whole = WT != 0 || c.C_out % (16 / static_cast<int>(sizeof(TIn))) == 0;
  if (fits && wfits && forced != Forced::kVec &&
      (by_pairs || forced == Forced::kSlab || !vec_first<TIn>(c.v, C_in, c.C_out, w_whole))) {
    Call cc = c;
    cc.x_bytes = static_cast<uint32_t>(xb);
    slab_entry<TIn, TOut>()(cc, WT, C_in, static_cast<uint32_t>(wb));
    return;
  }
  launch_vec<TIn, TOut, WT>(c, C_in);
}

template <int WT>
void run(const Call& c, int in_dt, int out_dt, int C_in) {
  const Forced forced = forced_path();
  bool done = false;
  if (forced != Forced::kVec) {
    done = out_dt == SPCONV_F32 ? try_mfma<float, WT>(c, in_dt, C_in)
                                : try_mfma<uint16_t, WT>(c, in_dt, C_in);
  }
  if (done) return;
  if (in_dt == SPCONV_F32 && out_dt == SPCONV_F32)
    launch_generic<float, float, WT>(c, C_in, forced);
  else if (in_dt == SPCONV_F32)
    launch_generic<float, uint16_t, WT>(c, C_in, forced);
  else if (out_dt == SPCONV_F32)
    launch_generic<uint16_t, float, WT>(c, C_in, forced);
  else
    launch_generic<uint16_t, uint16_t, WT>(c, C_in, forced);
}

}  // namespace
}  // namespace spc
