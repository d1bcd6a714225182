// Sparse pooling, the transposed rule book, and the weight / bias gradients
// on gfx950.
//
// Pooling (Section 3 defines max-pooling MP(f,s) and average-pooling AP(f,s)
// as variants of SC(.,.,f,s)): one lane per (output position, 16-byte chunk
// of channels) walks the offsets of the SC gather map in ascending order;
// MP starts from the zero vector and takes IEEE maxNum (exact in any dtype),
// AP sums in fp32 and divides by prod_j f_j once.
//
// Transposed rule book (Section 3: DC(.,.,f,s) inverts SC(.,.,f,s), same
// connections reversed; the SC input gradient runs the same reversed pairs),
// for books whose filter overlaps or whose extents the stride does not divide
// (the others run on the pair lists, see the end):
//   k_class_keys + radix sort  SC input rows ordered by their offset class
//                              x mod s (stable, so by row inside a class):
//                              with f = s every row of a class takes the same
//                              single offset, so 16-row blocks stay uniform
//   k_inverse                  position of every row in that order
//   k_fill_i32 + k_scatter_transpose
//                              G^T[i][q] = 1 + SC output row of the pair of R_i
//                              whose input row sits at position q (each
//                              (offset, input row) has at most one pair)
// The output-stationary forward kernels then run DC and the input gradients
// over this map.  When f = s an SC input row has at most one pair, and where
// all of them have theirs DC and the SC input gradient run over the rule
// book's own pair lists instead (the forward kernels with one offset, W^i
// chosen per tile of pairs): one launch, with no empty offsets to walk.
//
// Weight gradient dW^i = sum over the pairs of R_i of (input row)^T x (output
// gradient row): the output positions of the rule book's schedule are cut
// into chunks of up to 4096 positions, and chunk c of R_i is its pairs whose
// output lies in chunk c; one workgroup forms the fp32 partial product of a
// chunk for a tile of dW^i on the matrix cores (pairs gathered row-major into
// LDS and contracted there), and a second kernel
// adds the chunks of every entry in ascending chunk order.  The bias
// gradient sums the output-gradient rows in fixed row chunks the same way.
// No atomics anywhere: results are bitwise reproducible.
#include <algorithm>

#include "internal.h"

namespace spc {
namespace {

__device__ __forceinline__ float bf16f(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}
// fp32 -> bf16, round to nearest even; NaN stays NaN.
__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<uint16_t>(u >> 16);
}

template <typename T> struct IO;
template <> struct IO<float> {
  static constexpr int kVec = 4;
  __device__ static float ld(const float* p, int64_t i) { return p[i]; }
  __device__ static void st(float* p, int64_t i, float v) { p[i] = v; }
  __device__ static void ld16(const float* p, int64_t i, float* v) {
    const float4 q = *reinterpret_cast<const float4*>(p + i);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
  }
  __device__ static void st16(float* p, int64_t i, const float* v) {
    *reinterpret_cast<float4*>(p + i) = make_float4(v[0], v[1], v[2], v[3]);
  }
};
template <> struct IO<uint16_t> {
  static constexpr int kVec = 8;
  __device__ static float ld(const uint16_t* p, int64_t i) { return bf16f(p[i]); }
  __device__ static void st(uint16_t* p, int64_t i, float v) { p[i] = to_bf16(v); }
  __device__ static void ld16(const uint16_t* p, int64_t i, float* v) {
    const uint4 q = *reinterpret_cast<const uint4*>(p + i);
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[2 * e] = __uint_as_float(w[e] << 16);
      v[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
  }
  __device__ static void st16(uint16_t* p, int64_t i, const float* v) {
    uint4 q;
    q.x = to_bf16(v[0]) | (static_cast<uint32_t>(to_bf16(v[1])) << 16);
    q.y = to_bf16(v[2]) | (static_cast<uint32_t>(to_bf16(v[3])) << 16);
    q.z = to_bf16(v[4]) | (static_cast<uint32_t>(to_bf16(v[5])) << 16);
    q.w = to_bf16(v[6]) | (static_cast<uint32_t>(to_bf16(v[7])) << 16);
    *reinterpret_cast<uint4*>(p + i) = q;
  }
};

inline unsigned grid_of(int64_t n, int64_t cap = 65536) {
  int64_t b = (n + 255) / 256;
  if (b > cap) b = cap;
  return static_cast<unsigned>(b < 1 ? 1 : b);
}

// ---------------------------------------------------------------------------
// Pooling
// ---------------------------------------------------------------------------
// Thread = (output position, VEC channels).  The gather-map entries of 8
// offsets are loaded together, then their input rows (an absent neighbour
// reads row 0 and is not taken), so the loads of a batch are in flight at
// once instead of one offset after another behind a branch; the rows are
// taken in ascending offset order.
template <typename T, int VEC, bool MAX>
__global__ __launch_bounds__(256) void k_pool(const int32_t* __restrict__ gmap,
                                              const int32_t* __restrict__ perm, int64_t gstride,
                                              const DeviceHeader* __restrict__ hdr, int K,
                                              const T* __restrict__ x, T* __restrict__ y, int C) {
  constexpr int KB = 8;
  const int nch = C / VEC;
  const int64_t total = hdr->n_out * nch;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; idx < total;
       idx += stride) {
    const int64_t p = idx / nch;
    const int c0 = static_cast<int>(idx - p * nch) * VEC;
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.0f;   // MP: the zero vector; AP: empty sum
    for (int i0 = 0; i0 < K; i0 += KB) {
      int32_t g[KB];
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const int i = i0 + u < K ? i0 + u : K - 1;
        g[u] = gmap[i * gstride + p] - 1;
      }
#pragma unroll
      for (int u = 0; u < KB; ++u) g[u] = i0 + u < K ? g[u] : -1;
      float v[KB][VEC];
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const int64_t base = static_cast<int64_t>(g[u] >= 0 ? g[u] : 0) * C + c0;
        if constexpr (VEC == 1) {
          v[u][0] = IO<T>::ld(x, base);
        } else {
          IO<T>::ld16(x, base, v[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        if (g[u] < 0) continue;
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = MAX ? fmaxf(acc[e], v[u][e]) : acc[e] + v[u][e];
      }
    }
    if constexpr (!MAX) {
      const float k = static_cast<float>(K);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] = acc[e] / k;
    }
    const int64_t ob = static_cast<int64_t>(perm[p]) * C + c0;
    if constexpr (VEC == 1) {
      IO<T>::st(y, ob, acc[0]);
    } else {
      IO<T>::st16(y, ob, acc);
    }
  }
}

template <typename T, bool MAX>
void launch_pool(spconv_rulebook rb, const void* x, void* y, int C, hipStream_t st) {
  const bool vec = C % IO<T>::kVec == 0;
  const int64_t work = rb->n_cap * (vec ? C / IO<T>::kVec : C);
  if (vec)
    k_pool<T, IO<T>::kVec, MAX><<<grid_of(work), 256, 0, st>>>(
        rb->gmap, rb->perm, rb->gstride, rb->hdr, static_cast<int>(rb->K),
        static_cast<const T*>(x), static_cast<T*>(y), C);
  else
    k_pool<T, 1, MAX><<<grid_of(work), 256, 0, st>>>(
        rb->gmap, rb->perm, rb->gstride, rb->hdr, static_cast<int>(rb->K),
        static_cast<const T*>(x), static_cast<T*>(y), C);
}

// ---------------------------------------------------------------------------
// Transposed rule book
// ---------------------------------------------------------------------------
struct ClassGeom {
  int D;
  int32_t s[kMaxD];
  int64_t mult[kMaxD];   // class = sum_j (x_j mod s_j) mult_j, last dimension fastest
};

__global__ __launch_bounds__(256) void k_class_keys(const int32_t* __restrict__ coords, int64_t n,
                                                    ClassGeom g, uint64_t* __restrict__ keys,
                                                    int32_t* __restrict__ vals) {
  const int64_t r = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (r >= n) return;
  uint64_t c = 0;
  for (int j = 1; j < g.D; ++j)
    c += static_cast<uint64_t>(coords[r * g.D + j] % g.s[j]) * static_cast<uint64_t>(g.mult[j]);
  keys[r] = c;
  vals[r] = static_cast<int32_t>(r);
}

__global__ __launch_bounds__(256) void k_iota(int32_t* __restrict__ a, int64_t n) {
  const int64_t r = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (r < n) a[r] = static_cast<int32_t>(r);
}

__global__ __launch_bounds__(256) void k_inverse(const int32_t* __restrict__ perm, int64_t n,
                                                 int32_t* __restrict__ iperm) {
  const int64_t q = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (q < n) iperm[perm[q]] = static_cast<int32_t>(q);
}

__global__ __launch_bounds__(256) void k_fill_i32(int32_t* __restrict__ a, int32_t v, int64_t n) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t r = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; r < n; r += stride)
    a[r] = v;
}

__global__ void k_set_rows(DeviceHeader* h, int64_t n) {
  if (threadIdx.x == 0) {
    h->status = 0;
    h->n_out = n;
  }
}

// One lane per pair of the rule book (R_0 first); the pair's offset is found
// by a binary search of the offset table.
__global__ __launch_bounds__(256) void k_scatter_transpose(
    const int32_t* __restrict__ pairs, const int64_t* __restrict__ pair_off, int K,
    const int32_t* __restrict__ iperm, int32_t* __restrict__ tgmap, int64_t tgstride) {
  const int64_t total = pair_off[K];
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t e = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; e < total;
       e += stride) {
    int lo = 0, hi = K;            // pair_off[lo] <= e < pair_off[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) / 2;
      if (pair_off[mid] <= e) lo = mid; else hi = mid;
    }
    const int32_t a = pairs[2 * e], b = pairs[2 * e + 1];
    tgmap[lo * tgstride + iperm[a]] = b + 1;
  }
}

// ---------------------------------------------------------------------------
// Weight and bias gradients
// ---------------------------------------------------------------------------
// One partial covers bpc blocks of kBlock output positions (dw_plan).
constexpr int kSub = 64;           // pairs staged in LDS at a time
constexpr int64_t kRowChunk = 512; // rows per bias-gradient partial

// The (offset, chunk) of this workgroup and its pair range inside R_i, from
// the rule book's per-block bases (blk_base[i][b] = first pair of R_i whose
// output is in block b of kBlock positions).  Workgroup L runs on XCD L mod 8;
// the K offsets of one chunk go to one XCD, so that the rows they share
// (every output row of the chunk, and its neighbours) meet in that L2.
struct DwChunk {
  int i, c;
  int64_t start, end;      // pair range [start, end) relative to R_i
};
__device__ __forceinline__ bool dw_chunk(const int32_t* blk_base, const int64_t* pair_off,
                                         int64_t nblk, int K, int nchunk, int bpc, DwChunk* d) {
  const int L = blockIdx.x, xcd = L % 8, q = L / 8;
  d->c = xcd + 8 * (q / K);
  d->i = q % K;
  if (d->c >= nchunk) return false;
  const int64_t b0 = static_cast<int64_t>(d->c) * bpc, b1 = b0 + bpc;
  const int64_t k_i = pair_off[d->i + 1] - pair_off[d->i];
  d->start = blk_base[d->i * nblk + b0];
  d->end = b1 < nblk && d->c + 1 < nchunk ? blk_base[d->i * nblk + b1] : k_i;
  return true;
}

// Matrix-core partial products of dW^i (fp32 accumulation): grid (the
// (offset, chunk) pairs of dw_chunk; TC x TN tile of dW^i).  Per step 64
// pairs: their input rows and gradient rows (this tile's columns of each) are
// gathered into LDS row-major; the contraction runs over pairs, on 32x32
// products (32x32x16 bf16, 32x32x2 fp32).  The tile's 32x32 quadrants are
// dealt to the four waves; where there are fewer than four, the waves of one
// quadrant share each step's pairs and their sums are added in wave order at
// the end.  So every result is a fixed-order sum, and a wave holds 16
// accumulator registers (four workgroups share a compute unit, which hides
// the gathers' latency better than larger steps with fewer workgroups).
//   bf16: an operand fragment holds one channel of 8 consecutive pairs; it
//   comes from the row-major tile through gfx950's transposing LDS read (16
//   lanes read 4 pairs x 16 channels, each receives one channel of the 4
//   pairs).  fp32: one channel of one pair per lane, a plain 4-byte read.
// Columns past C_in / C_out are zero.  AL: rows are whole 16-byte pieces;
// otherwise single elements are loaded.
//
// Measured: fp32, 348,208 surface rows 32 x 32 3^3, 1,143 us with the vector
// ALU kernel this replaced (64x64 tiles whatever the widths); 165 us
// here.
// (MFMA floor 53 us, gathers 1 GB).  bf16, 902,504 surface rows 64 x 64 3^3:
// 256 us with 16x16x32 products and one set of tiles, 252 us with 32x32x16 and
// two.
// dbpart != NULL (VSC): the workgroups of the centre offset, whose pairs are
// every output row once, also sum the gradient rows (the bias gradient) with
// one more product per fragment, a fragment of ones times the staged rows, in
// the waves of the first channel quadrant; dbpart[chunk][n] receives the
// chunk's column sums.
typedef short dw_s4 __attribute__((ext_vector_type(4)));
typedef __bf16 dw_bf8 __attribute__((ext_vector_type(8)));
typedef float dw_f16 __attribute__((ext_vector_type(16)));
typedef unsigned dw_u4 __attribute__((ext_vector_type(4)));

// Element types: KS pairs per product; frag() reads channels c0 .. c0 + 31 of
// pairs p0 .. p0 + KS - 1 from a tile of W-channel rows; at() places 16-byte
// piece k of row r so that the rows of one read fall on different banks
// (256-byte bank period; narrow tiles are contiguous there already).
template <typename T> struct Dw;
template <> struct Dw<uint16_t> {
  static constexpr int KS = 16;
  typedef dw_bf8 Frag;
  template <int W> __device__ static int at(int row, int col) {
    const int k = W == 64 ? (col >> 3) ^ (((row >> 1) & 1) << 2) : col >> 3;
    return row * W + ((k << 3) | (col & 7));
  }
  template <int W> __device__ static Frag frag(const uint16_t* tile, int p0, int c0, int lane) {
    // lanes 16q + j: pairs p0 + 8 (q / 2) + j / 4 (+4 for the upper half),
    // channels c0 + 16 (q % 2) + 4 (j % 4) .. + 3
    const int j = lane & 15, q = lane >> 4;
    const int row = p0 + 8 * (q >> 1) + (j >> 2), col = c0 + 16 * (q & 1) + 4 * (j & 3);
    typedef __attribute__((address_space(3))) dw_s4 lds_s4;
    // generic -> LDS address-space conversion (the tile is a __shared__ array)
    lds_s4* lo = (lds_s4*)(const_cast<uint16_t*>(tile) + at<W>(row, col));
    lds_s4* hi = (lds_s4*)(const_cast<uint16_t*>(tile) + at<W>(row + 4, col));
    const dw_s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lo);
    const dw_s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(hi);
    typedef short s8 __attribute__((ext_vector_type(8)));
    const s8 v = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return __builtin_bit_cast(dw_bf8, v);
  }
  __device__ static Frag ones() {
    Frag f;
#pragma unroll
    for (int k = 0; k < 8; ++k) f[k] = static_cast<__bf16>(1.0f);
    return f;
  }
  __device__ static dw_f16 mma(Frag a, Frag b, dw_f16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <> struct Dw<float> {
  static constexpr int KS = 2;
  typedef float Frag;
  template <int W> __device__ static int at(int row, int col) {
    const int k = W == 64 ? (col >> 2) ^ ((row & 1) << 3) : col >> 2;
    return row * W + ((k << 2) | (col & 3));
  }
  template <int W> __device__ static Frag frag(const float* tile, int p0, int c0, int lane) {
    return tile[at<W>(p0 + (lane >> 5), c0 + (lane & 31))];
  }
  __device__ static Frag ones() { return 1.0f; }
  __device__ static dw_f16 mma(Frag a, Frag b, dw_f16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};

// The 16 bytes of columns c .. of row `row`, zero where ok is false or past
// `width` columns.  AL: one load (row 0, column 0 when not ok); the caller
// zeroes.  Otherwise element loads, each from a column that exists.
template <typename T, bool AL>
__device__ __forceinline__ dw_u4 dw_piece(const T* __restrict__ p, int64_t row, int64_t width,
                                          int c, bool ok) {
  if constexpr (AL) {
    return *reinterpret_cast<const dw_u4*>(p + (ok ? row * width + c : 0));
  } else {
    const int64_t base = ok ? row * width : 0;
    dw_u4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (sizeof(T) == 4) {
        const int e = c + q;
        const uint32_t u = __float_as_uint(p[base + (e < width ? e : 0)]);
        v[q] = e < width ? u : 0u;
      } else {
        const int e = c + 2 * q;
        const uint32_t lo = p[base + (e < width ? e : 0)];
        const uint32_t hi = p[base + (e + 1 < width ? e + 1 : 0)];
        v[q] = (e < width ? lo : 0u) | (e + 1 < width ? hi << 16 : 0u);
      }
    }
    return v;
  }
}

template <typename T, bool DC, int TC, int TN, bool AL>
__global__ __launch_bounds__(256, !AL ? 2 : (sizeof(T) == 4 && TC != TN ? 3 : 4)) void k_dw_mfma(
    const int32_t* __restrict__ pairs, const int64_t* __restrict__ pair_off,
    const int32_t* __restrict__ blk_base, int64_t nblk, const T* __restrict__ x,
    const T* __restrict__ dy, int C_in, int C_out, int K, int nchunk, int bpc,
    float* __restrict__ part, int centre, float* __restrict__ dbpart) {
  using E = Dw<T>;
  constexpr int STEP = kSub;
  constexpr int EPP = 16 / static_cast<int>(sizeof(T));   // elements per 16-byte piece
  constexpr int LX = TC / EPP, LG = TN / EPP;             // lanes per staged row
  constexpr int PX = STEP * LX / 256, PG = STEP * LG / 256;   // passes of 256 lanes
  static_assert(PX >= 1 && PG >= 1, "a step fills the workgroup");
  constexpr int NQ = (TC / 32) * (TN / 32);               // quadrants
  constexpr int NS = 4 / NQ;                              // waves per quadrant
  constexpr int GRP = STEP / E::KS;                       // products per step
  // staging tiles (and, at the end, the waves' sums) and a ring of the pairs
  // of four steps; two sets of tiles while four workgroups still fit a compute
  // unit (the rows of step t + 1 then need no barrier of their own)
  constexpr int kTiles = STEP * (TC + TN);
  constexpr int kSums = (NS - 1) * NQ * 1024 * 4, kTileBytes = kTiles * static_cast<int>(sizeof(T));
  constexpr int NB = kTileBytes <= 16384 ? 2 : 1;
  __shared__ __attribute__((aligned(16)))
  unsigned char s_buf[kSums > NB * kTileBytes ? kSums : NB * kTileBytes];
  __shared__ int2 s_pr[4][STEP];
  T* const s_t = reinterpret_cast<T*>(s_buf);         // buffer t % NB: x rows, then dy rows
  DwChunk dc_;
  if (!dw_chunk(blk_base, pair_off, nblk, K, nchunk, bpc, &dc_)) return;
  const int i = dc_.i, chunk = dc_.c;
  const int ntn = (C_out + TN - 1) / TN;
  const int c0 = (blockIdx.y / ntn) * TC, n0 = (blockIdx.y % ntn) * TN;
  const int64_t base = pair_off[i];
  const int64_t start = dc_.start, end = dc_.end;
  const int nsteps = static_cast<int>((end - start + STEP - 1) / STEP);
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  float* out = part + (static_cast<int64_t>(i) * nchunk + chunk) * C_in * C_out;
  const bool dbt = dbpart && i == centre && c0 == 0;    // this tile sums the bias gradient
  if (nsteps == 0) {                                   // no pair of R_i in this chunk
    for (int t = threadIdx.x; t < TC * TN; t += 256) {
      const int c = c0 + t / TN, n = n0 + t % TN;
      if (c < C_in && n < C_out) out[static_cast<int64_t>(c) * C_out + n] = 0.0f;
    }
    if (dbt && threadIdx.x < TN && n0 + threadIdx.x < C_out)
      dbpart[static_cast<int64_t>(chunk) * C_out + n0 + threadIdx.x] = 0.0f;
    return;
  }

  // Over steps of STEP pairs: at step t the pairs of step t + 3 are loaded
  // (threads 0..STEP-1, one each) and, after the products, put in the LDS ring;
  // the data rows of step t + 2 are gathered (their pairs from the ring) into
  // one of two register sets, the products of step t run on the LDS tiles, and
  // the rows of step t + 1 (the other set) are written to LDS.  Every load is
  // unconditional (pairs past the chunk read its first pair; rows past the
  // chunk and columns past C read row 0 / column 0 and are zeroed when
  // staged), so no load sits under a branch, and the issue order (the pair
  // before the rows) lets the in-order load counter keep the rows in flight
  // while the pair is waited on.
  const int npairs = static_cast<int>(end - start);
  const int chx = (threadIdx.x % LX) * EPP, chg = (threadIdx.x % LG) * EPP;
  const bool colx = c0 + chx < C_in, colg = n0 + chg < C_out;
  typedef dw_u4 RowsX[PX];
  typedef dw_u4 RowsG[PG];
  auto pair_load = [&](int t) __attribute__((always_inline)) -> int2 {
    const int e = t * STEP + (threadIdx.x < STEP ? threadIdx.x : 0);
    return *reinterpret_cast<const int2*>(pairs + 2 * (base + start + (e < npairs ? e : 0)));
  };
  auto pair_put = [&](int t, int2 v) __attribute__((always_inline)) {
    if (threadIdx.x < STEP) s_pr[t & 3][threadIdx.x] = v;
  };
  auto gather = [&](int t, RowsX& vx, RowsG& vg, uint32_t& ok) __attribute__((always_inline)) {
    ok = 0;
#pragma unroll
    for (int p = 0; p < PX; ++p) {
      const int r = p * (256 / LX) + threadIdx.x / LX;
      const int2 pr = s_pr[t & 3][r];
      // (input row, gradient row); DC reads its pairs backwards
      const bool o = t * STEP + r < npairs && colx;
      ok |= (o ? 1u : 0u) << p;
      vx[p] = dw_piece<T, AL>(x, DC ? pr.y : pr.x, C_in, c0 + chx, o);
    }
#pragma unroll
    for (int p = 0; p < PG; ++p) {
      const int r = p * (256 / LG) + threadIdx.x / LG;
      const int2 pr = s_pr[t & 3][r];
      const bool o = t * STEP + r < npairs && colg;
      ok |= (o ? 1u : 0u) << (8 + p);
      vg[p] = dw_piece<T, AL>(dy, DC ? pr.x : pr.y, C_out, n0 + chg, o);
    }
  };
  auto stage = [&](int t, const RowsX& vx, const RowsG& vg, uint32_t ok)
      __attribute__((always_inline)) {
    T* s_x = s_t + (t % NB) * kTiles;
    T* s_g = s_x + STEP * TC;
    const dw_u4 z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int p = 0; p < PX; ++p)
      *reinterpret_cast<dw_u4*>(
          &s_x[E::template at<TC>(p * (256 / LX) + threadIdx.x / LX, chx)]) =
          (ok >> p) & 1u ? vx[p] : z;
#pragma unroll
    for (int p = 0; p < PG; ++p)
      *reinterpret_cast<dw_u4*>(
          &s_g[E::template at<TN>(p * (256 / LG) + threadIdx.x / LG, chg)]) =
          (ok >> (8 + p)) & 1u ? vg[p] : z;
  };

  // wave -> quadrant (qc, qn) and share ks of every step's products
  const int quad = wave % NQ, ks = wave / NQ;
  const int qc = quad / (TN / 32) * 32, qn = quad % (TN / 32) * 32;
  dw_f16 acc, accb;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = accb[e] = 0.0f;
  const bool dbw = dbt && qc == 0;
  const typename E::Frag ones = E::ones();

  RowsX xa, xb;
  RowsG ga, gb;
  uint32_t oka = 0, okb = 0;
  pair_put(0, pair_load(0));
  pair_put(1, pair_load(1));
  pair_put(2, pair_load(2));
  __syncthreads();
  gather(0, xa, ga, oka);
  gather(1, xb, gb, okb);
  stage(0, xa, ga, oka);
  __syncthreads();
  // step t: the set holding step t + 1 is `nx`, the free set `fr`
  // (the gather of step t + 2 is issued even past the last step, as rows that
  // are all zeroed, so that the number of loads in flight never depends on t)
  auto step = [&](int t, RowsX& nxx, RowsG& nxg, uint32_t& nok, RowsX& frx, RowsG& frg,
                  uint32_t& fok) __attribute__((always_inline)) {
    const int2 pn = pair_load(t + 3);
    gather(t + 2, frx, frg, fok);
    const T* s_x = s_t + (t % NB) * kTiles;
    const T* s_g = s_x + STEP * TC;
#pragma unroll
    for (int g = 0; g < GRP / NS; ++g) {        // this wave's share of the pairs, in order
      const int p0 = (ks * (GRP / NS) + g) * E::KS;
      const typename E::Frag fa = E::template frag<TC>(s_x, p0, qc, lane);
      const typename E::Frag fb = E::template frag<TN>(s_g, p0, qn, lane);
      acc = E::mma(fa, fb, acc);
      if (dbw) accb = E::mma(ones, fb, accb);
    }
    if (NB == 1) __syncthreads();              // the tiles are read
    if (t + 1 < nsteps) stage(t + 1, nxx, nxg, nok);
    pair_put(t + 3, pn);
    __syncthreads();
  };
  int t = 0;
  for (; t + 1 < nsteps; t += 2) {
    step(t, xb, gb, okb, xa, ga, oka);
    step(t + 1, xa, ga, oka, xb, gb, okb);
  }
  if (t < nsteps) step(t, xb, gb, okb, xa, ga, oka);
  // the sums of a quadrant's waves, added in wave order (the tiles are free:
  // the last step ended with a barrier)
  if constexpr (NS > 1) {
    float* s_sum = reinterpret_cast<float*>(s_buf);
    auto add = [&](dw_f16& a) {
      if (ks > 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) s_sum[(((ks - 1) * NQ + quad) * 16 + e) * 64 + lane] = a[e];
      }
      __syncthreads();
      if (ks == 0) {
#pragma unroll
        for (int k = 0; k < NS - 1; ++k)
#pragma unroll
          for (int e = 0; e < 16; ++e) a[e] += s_sum[((k * NQ + quad) * 16 + e) * 64 + lane];
      }
      __syncthreads();
    };
    add(acc);
    if (dbt) add(accb);                        // workgroup-uniform
  }
  if (ks > 0) return;
  // lane (r, h) holds rows 8 (e / 4) + 4 h + e % 4, column r of its quadrant
  const int r = lane % 32, h = lane / 32;
  const int n = n0 + qn + r;
  if (n >= C_out) return;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int c = c0 + qc + 8 * (e / 4) + 4 * h + e % 4;
    if (c < C_in) out[static_cast<int64_t>(c) * C_out + n] = acc[e];
  }
  if (dbw && h == 0)                           // every row of accb holds the sums
    dbpart[static_cast<int64_t>(chunk) * C_out + n] = accb[0];
}

// Bias gradient, stage 2 (workgroups of k_dw_reduce past the weight's): 4
// columns per workgroup; lane (phase q of 64, column) adds chunk partials q,
// q + 64, ... eight loads at a time into 8 accumulators (by round), then the
// 64 phases are added in a fixed tree.
__device__ void db_reduce_block(const float* __restrict__ partb, int nchunks, int C_out,
                                float* __restrict__ db, int blk) {
  constexpr int kPh = 64, kCols = 4;
  __shared__ float s[kPh][kCols + 1];
  const int q = threadIdx.x / kCols, cn = threadIdx.x % kCols;
  const int n = blk * kCols + cn;
  float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (n < C_out) {
    int ch = q;
    for (; ch + 7 * kPh < nchunks; ch += 8 * kPh) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = partb[static_cast<int64_t>(ch + u * kPh) * C_out + n];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] += v[u];
    }
    for (int u = 0; ch < nchunks; ch += kPh, ++u)
      a[u] += partb[static_cast<int64_t>(ch) * C_out + n];
  }
  s[q][cn] = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
  __syncthreads();
  for (int h = kPh / 2; h >= 1; h >>= 1) {
    if (q < h) s[q][cn] += s[q + h][cn];
    __syncthreads();
  }
  if (q == 0 && n < C_out) db[n] = s[0][cn];
}

// dw[i][c][n] = sum over the chunks of R_i.  The chunks are split into S
// consecutive segments (S = 1, 2, 4 or 8, chosen on the host so that small
// weight tensors still fill the device); in a segment chunk ch goes to
// accumulator ch mod 8 and the 8 accumulators are added in a fixed tree; the
// segments' sums are added in a fixed tree through LDS.  Every order is
// fixed, so the result is reproducible.  A workgroup covers 256 / S
// consecutive elements; its threads with the same segment read consecutive
// elements of a partial.  Workgroups from nb_dw on reduce the bias
// gradient's partials instead (db_reduce_block).
__global__ __launch_bounds__(256) void k_dw_reduce(const float* __restrict__ part, int K,
                                                   int C_in, int C_out, int nch, int S,
                                                   float* __restrict__ dw, int64_t nb_dw,
                                                   const float* __restrict__ partb, int nrc,
                                                   float* __restrict__ db) {
  if (blockIdx.x >= nb_dw) {
    db_reduce_block(partb, nrc, C_out, db, static_cast<int>(blockIdx.x - nb_dw));
    return;
  }
  __shared__ float s_seg[256];
  const int64_t per = static_cast<int64_t>(C_in) * C_out;
  const int E = 256 / S;                       // elements per workgroup
  const int el = threadIdx.x % E, seg = threadIdx.x / E;
  const int64_t idx = blockIdx.x * static_cast<int64_t>(E) + el;
  const bool live = idx < K * per;
  const int L = (nch + S - 1) / S;
  const int c0 = seg * L < nch ? seg * L : nch;
  const int c1 = c0 + L < nch ? c0 + L : nch;
  float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (live) {
    const int i = static_cast<int>(idx / per);
    const int64_t rem = idx - i * per;
    const float* p = part + static_cast<int64_t>(i) * nch * per + rem;
    int ch = c0;
    for (; ch + 8 <= c1; ch += 8) {
#pragma unroll
      for (int j = 0; j < 8; ++j) a[j] += p[static_cast<int64_t>(ch + j) * per];
    }
    for (int j = 0; ch + j < c1; ++j) a[j] += p[static_cast<int64_t>(ch + j) * per];
  }
  s_seg[threadIdx.x] = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
  __syncthreads();
  for (int h = S / 2; h >= 1; h /= 2) {        // segment t += segment t + h, t < h
    if (seg < h) s_seg[threadIdx.x] += s_seg[threadIdx.x + h * E];
    __syncthreads();
  }
  if (seg == 0 && live) dw[idx] = s_seg[threadIdx.x];
}

// Bias gradient, stage 1: a chunk of kRowChunk rows per workgroup and up to
// 32 groups of 16 bytes of columns (grid.y covers wider rows); lane (row
// phase ph, column group cg) sums rows ph, ph + P, ... of the chunk (P the
// largest power of two that fits, loads issued 8 rows at a time), then the
// phases are added in a fixed tree through LDS.
template <typename T>
__global__ __launch_bounds__(256) void k_db_partial(const T* __restrict__ dy, int64_t rows,
                                                    int C_out, float* __restrict__ partb) {
  constexpr int V = IO<T>::kVec;
  __shared__ float s[256][V + 1];
  const int ngrp_all = (C_out + V - 1) / V;       // 16-byte column groups of a row
  const int g0 = blockIdx.y * 32;
  const int ngrp = ngrp_all - g0 < 32 ? ngrp_all - g0 : 32;
  int nph = 1;
  while (nph * 2 * ngrp <= 256) nph *= 2;         // row phases: a power of two
  const int ph = threadIdx.x / ngrp, cgp = g0 + threadIdx.x % ngrp;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kRowChunk;
  const int64_t r1 = r0 + kRowChunk < rows ? r0 + kRowChunk : rows;
  float acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) acc[e] = 0.0f;
  const bool vec = C_out % V == 0;
  auto row_vals = [&](int64_t r, float* v) {
    if (vec) {
      IO<T>::ld16(dy, r * C_out + cgp * V, v);
    } else {
#pragma unroll
      for (int e = 0; e < V; ++e)
        v[e] = cgp * V + e < C_out ? IO<T>::ld(dy, r * C_out + cgp * V + e) : 0.0f;
    }
  };
  if (ph < nph) {
    int64_t r = r0 + ph;
    for (; r + 7 * nph < r1; r += 8 * nph) {      // 8 rows in flight, added in row order
      float v[8][V];
#pragma unroll
      for (int u = 0; u < 8; ++u) row_vals(r + u * nph, v[u]);
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] += v[u][e];
    }
    for (; r < r1; r += nph) {
      float v[V];
      row_vals(r, v);
#pragma unroll
      for (int e = 0; e < V; ++e) acc[e] += v[e];
    }
  }
#pragma unroll
  for (int e = 0; e < V; ++e) s[threadIdx.x][e] = acc[e];
  __syncthreads();
  for (int h = nph / 2; h >= 1; h >>= 1) {        // phase p absorbs phase p + h
    if (ph < h) {
#pragma unroll
      for (int e = 0; e < V; ++e) s[threadIdx.x][e] += s[threadIdx.x + h * ngrp][e];
    }
    __syncthreads();
  }
  if (ph == 0) {
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const int n = cgp * V + e;
      if (n < C_out) partb[static_cast<int64_t>(blockIdx.x) * C_out + n] = s[threadIdx.x][e];
    }
  }
}


// How the output positions are cut into partials: bpc blocks of kBlock
// positions each, at most 16 (4096 positions: a row the K offsets share comes
// back while it is in L2).  Fewer shorten the steps of the fullest chunk, which
// bound layers with few chunks; more keep the partials small, which are written
// and read once.  The plan takes the bpc whose estimate is least (us; fitted to
// 712 layers of 490 to 345,353 rows, 1 to 27 offsets, both types, every bpc
// timed: within 2.3 % of each layer's best on average, where halving bpc until
// 4096 workgroups were reached was 8 % off; 345,353 rows K = 1 bf16 128 -> 128:
// 44 / 66 us with 8 / 4 blocks; 48,184 rows of a strided 3^3 24 -> 40: 22 / 37
// with 8 / 1; 3,305 pen rows 3^2 fp32 24 -> 40: 14 / 87 with 1 / 16), below 16
// only while the partials stay within 32 MB.
//   fill     pairs per offset and output position: n_in / (n_out prod s) of an
//            SC book; half the offsets other than the centre of a VSC book
//   step     one step of kSub pairs; the narrower tiles' is 0.3 of it
//   750      workgroups at work at a time
// The row counts are the host's best knowledge, so a book's plan may change
// when it is synchronised; the workspace query and the gradient both
// synchronise first.
struct DwPlan {
  int nchunk, bpc, tc, tn;
};
DwPlan dw_plan(spconv_rulebook rb, int dt, int C_in, int C_out) {
  DwPlan p;
  p.tc = C_in <= 32 ? 32 : 64;
  p.tn = C_out <= 32 ? 32 : 64;
  const int64_t rows = rb->synced && rb->n_out < rb->n_cap ? rb->n_out : rb->n_cap;
  const int64_t nblk = (rows + kBlock - 1) / kBlock;
  const int64_t tiles = static_cast<int64_t>((C_in + p.tc - 1) / p.tc) *
                        ((C_out + p.tn - 1) / p.tn);
  const int64_t per = 4ll * C_in * C_out * rb->K;        // bytes of one chunk's partials
  double strides = 1.0;
  for (int j = 1; j < rb->D; ++j) strides *= rb->s[j];
  const bool vsc = rb->kind == SPCONV_VSC;
  const double full = vsc || rows == 0 ? 1.0
                                       : std::min(1.0, static_cast<double>(rb->n_in) /
                                                           (strides * static_cast<double>(rows)));
  const double fill = vsc && rb->K > 1 ? 0.5 : full;
  const double step = (dt == SPCONV_F32 ? 3.0 : 0.57) * (p.tc + p.tn == 128 ? 1.0 : 0.3);
  // chunks that one thread of the reduction adds in turn (see its launch)
  const double segs = std::min(8.0, std::max(1.0, 131072.0 * 4.0 / static_cast<double>(per)));
  constexpr double kSteps = static_cast<double>(kBlock) / kSub;     // of a full block
  p.bpc = 16;
  double best = 0.0;
  for (int b = 16; b >= 1; b /= 2) {
    const int64_t nchunk = (nblk + b - 1) / b;
    if (b < 16 && per * nchunk > (32ll << 20)) break;
    const double blocks = static_cast<double>(std::min<int64_t>(b, nblk));
    const double nc = static_cast<double>(nchunk);
    const double chain = kSteps * blocks * full * step;
    const double work = static_cast<double>(rb->K * tiles) * nc *
                        std::max(2.35, kSteps * blocks * fill) * step / 750.0;
    const double t = std::max(chain, work) + 0.33 * std::min(chain, work) +
                     0.37e-6 * static_cast<double>(per) * nc + 0.068 * nc / segs;
    if (b == 16 || t < best) {
      best = t;
      p.bpc = b;
    }
  }
  p.nchunk = static_cast<int>((nblk + p.bpc - 1) / p.bpc);
  return p;
}

template <typename T, int TC, int TN>
void launch_dw(spconv_rulebook rb, const DwPlan& p, bool dc, const void* x, const void* dy,
               int C_in, int C_out, float* part, int centre, float* dbpart, hipStream_t st) {
  constexpr int EPP = 16 / static_cast<int>(sizeof(T));
  const int K = static_cast<int>(rb->K);
  const int tiles = ((C_in + TC - 1) / TC) * ((C_out + TN - 1) / TN);
  // (offset, chunk) pairs: 8 XCDs x K offsets x ceil(nchunk / 8) chunks each
  const dim3 grid(static_cast<unsigned>(8 * K * ((p.nchunk + 7) / 8)),
                  static_cast<unsigned>(tiles));
  // C % EPP == 0 keeps every gathered 16-byte load inside its row
  const bool al = C_in % EPP == 0 && C_out % EPP == 0;
  auto kern = al ? (dc ? k_dw_mfma<T, true, TC, TN, true> : k_dw_mfma<T, false, TC, TN, true>)
                 : (dc ? k_dw_mfma<T, true, TC, TN, false> : k_dw_mfma<T, false, TC, TN, false>);
  kern<<<grid, 256, 0, st>>>(rb->pairs, rb->pair_off, rb->blk_cnt, rb->nblk,
                             static_cast<const T*>(x), static_cast<const T*>(dy), C_in, C_out, K,
                             p.nchunk, p.bpc, part, centre, dbpart);
}

template <typename T>
void launch_dw_tile(spconv_rulebook rb, const DwPlan& p, bool dc, const void* x, const void* dy,
                    int C_in, int C_out, float* part, int centre, float* dbpart,
                    hipStream_t st) {
  auto f = p.tc == 32 ? (p.tn == 32 ? launch_dw<T, 32, 32> : launch_dw<T, 32, 64>)
                      : (p.tn == 32 ? launch_dw<T, 64, 32> : launch_dw<T, 64, 64>);
  f(rb, p, dc, x, dy, C_in, C_out, part, centre, dbpart, st);
}

}  // namespace

// ---------------------------------------------------------------------------
// Host entry points (called by abi.hip after argument checks)
// ---------------------------------------------------------------------------
int pool_forward(spconv_rulebook rb, int mode, int dt, const void* x, void* y, int C,
                 hipStream_t st) {
  if (rb->n_cap == 0) return SPCONV_OK;
  if (dt == SPCONV_F32) {
    if (mode == SPCONV_POOL_MAX) launch_pool<float, true>(rb, x, y, C, st);
    else launch_pool<float, false>(rb, x, y, C, st);
  } else {
    if (mode == SPCONV_POOL_MAX) launch_pool<uint16_t, true>(rb, x, y, C, st);
    else launch_pool<uint16_t, false>(rb, x, y, C, st);
  }
  return hipGetLastError() == hipSuccess ? SPCONV_OK : SPCONV_EHIP;
}

size_t transpose_bytes(int64_t n_in, int64_t K) {
  const int64_t tgstride = ((n_in + kBlock - 1) / kBlock) * kBlock;
  auto al = [](size_t v) { return (v + 255) / 256 * 256; };
  return al(256) + al(static_cast<size_t>(n_in) * 4) + al(static_cast<size_t>(K * tgstride) * 4);
}

int build_transpose(spconv_rulebook rb, const int32_t* coords, char* mem) {
  const int64_t n = rb->n_in;
  auto al = [](size_t v) { return (v + 255) / 256 * 256; };
  rb->t_hdr = reinterpret_cast<DeviceHeader*>(mem);
  rb->t_perm = reinterpret_cast<int32_t*>(mem + al(256));
  rb->t_gstride = ((n + kBlock - 1) / kBlock) * kBlock;
  rb->t_gmap = reinterpret_cast<int32_t*>(mem + al(256) + al(static_cast<size_t>(n) * 4));
  hipStream_t st = rb->stream;
  k_set_rows<<<1, 64, 0, st>>>(rb->t_hdr, n);
  k_fill_i32<<<grid_of(rb->K * rb->t_gstride), 256, 0, st>>>(rb->t_gmap, 0, rb->K * rb->t_gstride);
  if (n == 0) return hipGetLastError() == hipSuccess ? SPCONV_OK : SPCONV_EHIP;

  ClassGeom g{};
  g.D = rb->D;
  int64_t classes = 1;
  for (int j = rb->D - 1; j >= 1; --j) {
    g.s[j] = rb->s[j];
    g.mult[j] = classes;
    classes *= rb->s[j];
  }
  const size_t scratch = radix_sort_scratch_bytes(n);
  const size_t tbytes = 2 * al(static_cast<size_t>(n) * 8) + 3 * al(static_cast<size_t>(n) * 4) +
                        al(scratch);
  void* tmem = nullptr;
  if (dev_alloc(rb, tbytes, st, &tmem) != SPCONV_OK) return SPCONV_ENOMEM;
  char* p = static_cast<char*>(tmem);
  uint64_t* keys = reinterpret_cast<uint64_t*>(p);
  uint64_t* keys_tmp = reinterpret_cast<uint64_t*>(p + al(n * 8));
  int32_t* vals = reinterpret_cast<int32_t*>(p + 2 * al(n * 8));
  int32_t* vals_tmp = reinterpret_cast<int32_t*>(p + 2 * al(n * 8) + al(n * 4));
  int32_t* iperm = reinterpret_cast<int32_t*>(p + 2 * al(n * 8) + 2 * al(n * 4));
  void* sort_scratch = p + 2 * al(n * 8) + 3 * al(n * 4);
  if (classes > 1) {
    k_class_keys<<<grid_of(n, 1ll << 30), 256, 0, st>>>(coords, n, g, keys, vals);
    const bool flipped = radix_sort_pairs(keys, vals, keys_tmp, vals_tmp, rb->t_hdr, n,
                                          bitlen(static_cast<uint64_t>(classes - 1)), sort_scratch,
                                          st);
    if (hipMemcpyAsync(rb->t_perm, flipped ? vals_tmp : vals, static_cast<size_t>(n) * 4,
                       hipMemcpyDeviceToDevice, st) != hipSuccess) {
      (void)hipGetLastError();
      (void)dev_free(rb, tmem, st);
      return SPCONV_EHIP;
    }
  } else {
    k_iota<<<grid_of(n, 1ll << 30), 256, 0, st>>>(rb->t_perm, n);
  }
  k_inverse<<<grid_of(n, 1ll << 30), 256, 0, st>>>(rb->t_perm, n, iperm);
  k_scatter_transpose<<<grid_of(rb->K * n), 256, 0, st>>>(rb->pairs, rb->pair_off,
                                                          static_cast<int>(rb->K), iperm,
                                                          rb->t_gmap, rb->t_gstride);
  if (dev_free(rb, tmem, st) != SPCONV_OK) return SPCONV_EHIP;
  return hipGetLastError() == hipSuccess ? SPCONV_OK : SPCONV_EHIP;
}

// The reversed direction of an SC book (DC, the SC input gradient).  Where f =
// s and every SC input row has its pair it runs over the pair lists.  The
// extents may say so (t_direct); otherwise rows near the far border may lack
// theirs (their output site falls off the SC grid), and the pair total tells
// (read once, a wait).  All other books walk the transposed map.
int reversed_view(spconv_rulebook rb, FwdView* out) {
  bool paired = rb->t_direct;
  if (!paired && rb->n_in > 0) {
    paired = true;
    for (int j = 1; j < rb->D; ++j) paired = paired && rb->f[j] == rb->s[j];
  }
  if (paired && !rb->t_direct) {
    if (rb->h_total < 0) {
      int64_t total = 0;
      if (hipMemcpyAsync(&total, rb->pair_off + rb->K, sizeof(int64_t), hipMemcpyDeviceToHost,
                         rb->stream) != hipSuccess ||
          hipStreamSynchronize(rb->stream) != hipSuccess) {
        (void)hipGetLastError();
        return SPCONV_EHIP;
      }
      rb->h_total = total;
    }
    paired = rb->h_total == rb->n_in;
  }
  FwdView v{};
  v.n_cap = rb->n_in;
  v.n_src = rb->n_cap;
  if (paired) {
    v.hdr = rb->hdr;
    v.K = 1;
    v.K_row = 1;
    v.pairs = rb->pairs;
    v.pair_off = rb->pair_off;
    v.pair_K = static_cast<int>(rb->K);
  } else {
    v.gmap = rb->t_gmap;
    v.perm = rb->t_perm;
    v.gstride = rb->t_gstride;
    v.hdr = rb->t_hdr;
    v.K = rb->K;
    v.K_row = 1;                          // an input row's class takes every s-th offset
    for (int j = 1; j < rb->D; ++j) v.K_row *= (rb->f[j] + rb->s[j] - 1) / rb->s[j];
  }
  *out = v;
  return SPCONV_OK;
}

size_t backward_weight_workspace(spconv_rulebook rb, int C_in, int C_out, int op) {
  const int64_t rows = op == SPCONV_OP_DC ? rb->n_in : rb->n_cap;
  const int64_t nrc = (rows + kRowChunk - 1) / kRowChunk;
  // the query does not name the type: room for either plan
  const int64_t nchunk = std::max(dw_plan(rb, SPCONV_F32, C_in, C_out).nchunk,
                                  dw_plan(rb, SPCONV_BF16, C_in, C_out).nchunk);
  const int64_t nb = nrc > nchunk ? nrc : nchunk;      // rows of the bias partials
  return static_cast<size_t>(rb->K * nchunk) * C_in * C_out * 4 +
         static_cast<size_t>(nb > 0 ? nb : 1) * C_out * 4 + 256;
}

int backward_weight(spconv_rulebook rb, int op, int dt, const void* x, const void* dy, float* dw,
                    float* db, int C_in, int C_out, void* ws, hipStream_t st) {
  const DwPlan plan = dw_plan(rb, dt, C_in, C_out);
  const int nchunk = plan.nchunk;
  const int K = static_cast<int>(rb->K);
  float* part = static_cast<float*>(ws);
  const int64_t per = static_cast<int64_t>(C_in) * C_out;
  // VSC: the bias gradient comes from the weight gradient's centre-offset
  // workgroups (its pairs are every output row once, each with itself), per
  // chunk, into the bias partials' area (at least nchunk rows of C_out floats)
  int centre = 0;
  for (int j = 0; j < rb->D; ++j) centre = centre * rb->f[j] + (rb->f[j] - 1) / 2;
  const bool db_fused = db && op == SPCONV_OP_VSC && nchunk > 0;
  float* partb_fused = part + static_cast<int64_t>(rb->K) * nchunk * per;
  if (nchunk > 0)
    (dt == SPCONV_F32 ? launch_dw_tile<float> : launch_dw_tile<uint16_t>)(
        rb, plan, op == SPCONV_OP_DC, x, dy, C_in, C_out, part, db_fused ? centre : -1,
        db_fused ? partb_fused : nullptr, st);
  // bias-gradient partials: from k_dw_mfma (fused) or one pass over dy
  const float* partb = nullptr;
  int nrc = 0;
  if (db_fused) {
    partb = partb_fused;
    nrc = static_cast<int>(nchunk);
  } else if (db) {
    const int64_t rows = op == SPCONV_OP_DC ? rb->n_in : rb->n_out;
    nrc = static_cast<int>((rows + kRowChunk - 1) / kRowChunk);
    float* pb = part + static_cast<int64_t>(rb->K) * nchunk * per;
    partb = pb;
    if (nrc > 0) {
      const int vec = dt == SPCONV_F32 ? 4 : 8;
      const int groups = (C_out + vec - 1) / vec;
      dim3 g(static_cast<unsigned>(nrc), static_cast<unsigned>((groups + 31) / 32));
      if (dt == SPCONV_F32)
        k_db_partial<float><<<g, 256, 0, st>>>(static_cast<const float*>(dy), rows, C_out, pb);
      else
        k_db_partial<uint16_t><<<g, 256, 0, st>>>(static_cast<const uint16_t*>(dy), rows, C_out,
                                                  pb);
    }
  }
  {
    // one launch sums both: the weight's elements, then the bias columns.
    // Segments per weight element: enough threads for the device (~128 K),
    // at least 8 chunks per segment (more segments did not speed up the
    // headline's 95 MB of partials)
    const int64_t elems = static_cast<int64_t>(rb->K) * per;
    int S = 1;
    while (S < 8 && elems * S < (int64_t{1} << 17) && nchunk / (2 * S) >= 8) S *= 2;
    const int64_t E = 256 / S;
    const int64_t nb_dw = (elems + E - 1) / E;
    const int64_t nb_db = db ? (C_out + 3) / 4 : 0;
    if (nb_dw + nb_db > 0)
      k_dw_reduce<<<static_cast<unsigned>(nb_dw + nb_db), 256, 0, st>>>(
          part, K, C_in, C_out, nchunk, S, dw, nb_dw, partb, nrc, db);
  }
  return hipGetLastError() == hipSuccess ? SPCONV_OK : SPCONV_EHIP;
}

}  // namespace spc
