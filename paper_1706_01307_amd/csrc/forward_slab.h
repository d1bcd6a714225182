// Matrix-core forward for channel counts outside k_fwd_mfma's set (one object
// file per pair of element types).
#pragma once

#include "forward_kernels.h"

namespace spc {
namespace {

// ---------------------------------------------------------------------------
// Matrix-core path for any channel counts
// ---------------------------------------------------------------------------
// k_fwd_slab: the same output-stationary multiply-add as k_fwd_mfma, for input
// rows of any width.  The contraction of an offset is cut into slabs of
// SLAB = NCH k-chunks of channels (64 bf16 or 32 fp32 for NCH = 2), and the
// kernel walks the (offset, slab) steps in order, so the registers and the LDS
// image of W hold one slab however wide the rows are, and a tile keeps up to
// 128 output columns (every gathered row is then read once per 128 columns).
// Channels past C_in are zeros on both sides (buffer loads out of range),
// columns past C_out are computed on zeros and not stored.
//
// Bound: as k_fwd_mfma by the gathers and the per-step latency; these widths
// ran one lane per output column before, a serial chain of K C_in loads and
// multiply-adds (87,052 surface rows 192 -> 96 bf16 3^3 with the epilogue:
// 7,960 us, now 167 us; 64 CAD grids of 32^3, 24 -> 40 fp32 3^3 stride 2, the
// whole layer with its book: 297 us, now 94 us).  AX / AW: whether the rows of
// x (and W^T) / of W are whole 16-byte pieces; otherwise single elements are
// loaded, which needs no alignment beyond the element's.
template <typename TIn> __device__ __forceinline__ uint32_t buf_elem(__amdgpu_buffer_rsrc_t r,
                                                                     uint32_t off) {
  if constexpr (sizeof(TIn) == 4)
    return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
  else
    return __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
}

// 16 bytes at byte `off` (kBufOOB: zeros), of which the first `n` elements
// exist; one 16-byte load when AL, else element by element.
template <typename TIn, bool AL>
__device__ __forceinline__ u32x4 buf_piece(__amdgpu_buffer_rsrc_t r, uint32_t off, int n) {
  constexpr int ESZ = static_cast<int>(sizeof(TIn));
  if constexpr (AL) {
    return buf_load16(r, n > 0 ? off : kBufOOB);
  } else {
    u32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if constexpr (ESZ == 4) {
        v[q] = buf_elem<TIn>(r, q < n ? off + q * 4 : kBufOOB);
      } else {
        const uint32_t a = buf_elem<TIn>(r, 2 * q < n ? off + q * 4 : kBufOOB);
        const uint32_t b = buf_elem<TIn>(r, 2 * q + 1 < n ? off + q * 4 + 2 : kBufOOB);
        v[q] = a | (b << 16);
      }
    }
    return v;
  }
}

// Staging of one slab of W^i (SLAB k-rows, COLS columns from col0) into its
// LDS image, transposed as WImage describes.  WT 0: a task is KPT k-rows x one
// 16-byte piece of columns (bf16 packs pairs of k-rows); WT 1 / 2 (w holds
// W^T): one 16-byte piece of k of one column.
template <typename TIn, typename TOut, int NCH, int NCB, int WT, bool AX, bool AW>
struct WStage {
  static constexpr int ESZ = static_cast<int>(sizeof(TIn));
  static constexpr int EPP = 16 / ESZ;
  static constexpr int SLAB = NCH * MT<TIn>::KC;
  static constexpr int COLS = NCB * 16;
  static constexpr int ROWB = SLAB * ESZ;
  static constexpr int KPT = ESZ == 2 ? 2 : 1;
  static constexpr int NGRP = COLS / EPP;
  static constexpr int CPR = ROWB / 16;
  static constexpr int NTASK = WT == 0 ? (SLAB / KPT) * NGRP : COLS * CPR;
  static constexpr int TPT = (NTASK + 255) / 256;
  static constexpr int NWR = WT == 0 ? TPT * KPT : TPT;
  typedef u32x4 Regs[NWR];

  // slab of channels c0 .. of w[iv]; zeros where `in` is false
  __device__ static void load(__amdgpu_buffer_rsrc_t wr, bool in, int iv, int c0, int C_in,
                              int C_out, int col0, Regs& r) {
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
      const int t = threadIdx.x + q * 256;
      const bool live = in && (NTASK % 256 == 0 || t < NTASK);
      if constexpr (WT == 0) {
        const int k = c0 + t / NGRP * KPT, n = col0 + t % NGRP * EPP;
#pragma unroll
        for (int e = 0; e < KPT; ++e) {
          const int cnt = live && k + e < C_in ? C_out - n : 0;
          const uint32_t off = ((static_cast<uint32_t>(iv) * C_in + k + e) * C_out + n) * ESZ;
          r[q * KPT + e] = buf_piece<TIn, AW>(wr, off, cnt);
        }
      } else {
        const int n = col0 + t / CPR, k = c0 + t % CPR * EPP;
        const int cnt = live && n < C_out ? C_in - k : 0;
        const uint32_t off = ((static_cast<uint32_t>(iv) * C_out + n) * C_in + k) * ESZ;
        r[q] = buf_piece<TIn, AX>(wr, off, cnt);
      }
    }
  }
  __device__ static int row_of(int n) { return TileCols<TIn, TOut, NCB, true>::row_of(n); }
  __device__ static void store(unsigned char* dst, const Regs& r) {
#pragma unroll
    for (int q = 0; q < TPT; ++q) {
      const int t = threadIdx.x + q * 256;
      if (NTASK % 256 != 0 && t >= NTASK) continue;
      if constexpr (WT == 0) {
        const int kt = t / NGRP, nt = t % NGRP;
#pragma unroll
        for (int j = 0; j < EPP; ++j) {
          uint32_t v;
          if constexpr (ESZ == 2) {
            const uint32_t a = r[q * KPT][j / 2], b = r[q * KPT + 1][j / 2];
            v = (j & 1) ? ((a >> 16) | (b & 0xffff0000u)) : ((a & 0xffffu) | (b << 16));
          } else {
            v = r[q][j];
          }
          *reinterpret_cast<uint32_t*>(&dst[WImage<TIn, ROWB>::at(row_of(nt * EPP + j), kt * 4)]) = v;
        }
      } else {
        const int n = t / CPR, kc = t % CPR;
        *reinterpret_cast<u32x4*>(&dst[WImage<TIn, ROWB>::at(row_of(n), kc * 16)]) = r[q];
      }
    }
  }
};

// Whether any of the lane's sums is an infinity or NaN.
template <int RB, int NCB>
__device__ __forceinline__ bool nonfinite(const f32x4 (&acc)[RB][NCB]) {
  float z = 0.0f;
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) z = fmaf(acc[b][cb][v], 0.0f, z);
  return z != z;
}

// A row that lacks offset i enters the products of its 16-row block as zeros,
// and 0 times a non-finite W^i is NaN, where the row has no term at all.  So a
// wave that ends with a non-finite sum adds its tile up again over the rows'
// own pairs, one element per lane at a time as k_fwd_vec does.
template <typename TIn, typename TOut, int WT>
__device__ __forceinline__ void sum_over_pairs(
    const int32_t* gmap, const int32_t* perm, int64_t gstride, int64_t n_rows, int K,
    const TIn* x, const TIn* w, const float* bias, TOut* y, int C_in, int C_out, int64_t row0,
    int rows, int col0, int cols, const Epilogue& epi) {
  for (int e = __lane_id(); e < rows * cols; e += kWave) {
    const int64_t p = row0 + e / cols;
    const int col = col0 + e % cols;
    if (p >= n_rows || col >= C_out) continue;
    float acc = 0.0f;
    for (int i = 0; i < K; ++i) {
      const int64_t g = static_cast<int64_t>(gmap[i * gstride + p]) - 1;
      if (g < 0) continue;
      for (int c = 0; c < C_in; ++c)
        acc = fmaf(ElemIO<TIn>::load(x, g * C_in + c),
                   ElemIO<TIn>::load(w, w_index<WT>(i, K, c, col, C_in, C_out)), acc);
    }
    store_elem(acc, static_cast<int64_t>(perm[p]) * C_out + col, col, bias, epi, y);
  }
}

// PAIRS: a pair view (K = 1), from which the tile's rows and its W^i come, in
// the arguments of the map, the schedule and K.
template <typename TIn, typename TOut, int NCH, int NCB, int RB, int WT, bool AX, bool AW,
          bool PAIRS>
__global__ __launch_bounds__(256, 2) void k_fwd_slab(
    const int32_t* __restrict__ gmap, const int32_t* __restrict__ perm, int64_t gstride,
    const DeviceHeader* __restrict__ hdr, int K_arg, const TIn* __restrict__ x, uint32_t x_bytes,
    const TIn* __restrict__ w, uint32_t w_bytes, const float* __restrict__ bias,
    TOut* __restrict__ y, int C_in, int C_out, int64_t ntiles, Epilogue epi) {
  const int K = PAIRS ? 1 : K_arg;
  constexpr int KC = MT<TIn>::KC;
  constexpr int SLAB = NCH * KC;
  constexpr int COLS = NCB * 16;
  constexpr int ESZ = static_cast<int>(sizeof(TIn));
  constexpr int EPP = 16 / ESZ;                   // elements per 16-byte piece
  constexpr int ROWB = SLAB * ESZ;                // bytes of one row's slab
  constexpr int WAVE_ROWS = RB * 16;
  constexpr int TILE_ROWS = 4 * WAVE_ROWS;

  __shared__ __attribute__((aligned(16))) unsigned char s_w[2][WImage<TIn, ROWB>::bytes(COLS)];

  // XCD-contiguous tile ranges over the device-side row count, as k_fwd_mfma
  PairTile pt{0, 0, 0};
  int64_t n_rows = TILE_ROWS, tile = 0;
  if constexpr (PAIRS) {
    if (!pair_tile<TILE_ROWS>(reinterpret_cast<const int64_t*>(perm), K_arg, ntiles, &pt)) return;
  } else {
    n_rows = hdr->n_out;
    const int64_t nt_real = (n_rows + TILE_ROWS - 1) / TILE_ROWS;
    const int64_t nt = nt_real < ntiles ? nt_real : ntiles;
    const int64_t per = (nt + 7) / 8;
    const int64_t q8 = blockIdx.x / 8;
    if (q8 >= per) return;
    tile = static_cast<int64_t>(blockIdx.x % 8) * per + q8;
    if (tile >= nt) return;
  }

  const int col0 = blockIdx.y * COLS;
  const int wave = threadIdx.x / kWave;
  const int uwave = __builtin_amdgcn_readfirstlane(wave);   // (a scalar: no register kept)
  const int lane = threadIdx.x % kWave;
  const int lr = lane % 16, lg = lane / 16;
  const int64_t row0 = tile * TILE_ROWS + wave * WAVE_ROWS;
  const uint32_t row_bytes = static_cast<uint32_t>(C_in) * ESZ;
  const __amdgpu_buffer_rsrc_t xr = buf_rsrc(x, x_bytes);
  const __amdgpu_buffer_rsrc_t wr_ = buf_rsrc(w, w_bytes);
  const uint32_t gmap_bytes = static_cast<uint32_t>(gstride * 4);

  // The (offset, slab) of a step, advanced one step at a time (i = K: past
  // the last step, everything reads zeros).
  const int nslab = (C_in + SLAB - 1) / SLAB;
  struct At { int i, c; };                        // offset, first channel of the slab
  auto next = [&](At& a) {
    a.c += SLAB;
    if (a.c >= C_in) {
      a.c = 0;
      ++a.i;
    }
  };

  using WS = WStage<TIn, TOut, NCH, NCB, WT, AX, AW>;
  typedef typename WS::Regs WRegs;
  auto w_load = [&](At a, WRegs& r) {
    const int iv = PAIRS ? pt.i : (WT == 1 ? K - 1 - a.i : a.i);
    WS::load(wr_, a.i < K, iv, a.c, C_in, C_out, col0, r);
  };
  auto w_store = [&](int buf, const WRegs& r) { WS::store(s_w[buf], r); };

  typedef int32_t GRegs;
  const int64_t map_row = row0 + map_lane<RB>(lane);
  const uint32_t map_off = map_row < n_rows ? static_cast<uint32_t>(map_row) * 4u : kBufOOB;
  auto g_load = [&](At a, GRegs& g) {
    if constexpr (PAIRS) {
      g = pair_row(gmap, pt, static_cast<int>(map_row), 1);
      return;
    }
    const int ic = a.i < K ? a.i : 0;
    const __amdgpu_buffer_rsrc_t gr = buf_rsrc(gmap + static_cast<int64_t>(ic) * gstride,
                                               gmap_bytes);
    g = static_cast<int32_t>(__builtin_amdgcn_raw_buffer_load_b32(
            gr, a.i < K ? map_off : kBufOOB, 0, 0)) - 1;
  };
  typedef u32x4 ARegs[RB][NCH];
  auto a_load = [&](At at, const GRegs& gv, ARegs& a) -> uint32_t {
    int32_t g[RB];
    spread_map<RB>(gv, g);
#pragma unroll
    for (int b = 0; b < RB; ++b) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        const int c = at.c + ch * KC + lg * EPP;
        const int cnt = g[b] >= 0 ? C_in - c : 0;
        const uint32_t off = static_cast<uint32_t>(g[b]) * row_bytes + static_cast<uint32_t>(c) * ESZ;
        a[b][ch] = buf_piece<TIn, AX>(xr, off, cnt);
      }
    }
    return map_blocks<RB>(gv);
  };

  f32x4 acc[RB][NCB];
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[b][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto mma = [&](At at, int buf, const ARegs& a, uint32_t pres) {
    const unsigned char* sw = s_w[buf];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      if (ch > 0 && at.c + ch * KC >= C_in) break;       // chunks past the rows' end
      u32x4 bw[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
        bw[cb] = *reinterpret_cast<const u32x4*>(
            &sw[WImage<TIn, ROWB>::at(cb * 16 + lr, ch * 64 + lg * 16)]);
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        if (!(pres & (1u << b))) continue;               // all 16 rows lack this offset
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[b][cb] = MT<TIn>::mma(bw[cb], a[b][ch], acc[b][cb]);
      }
    }
  };

  // The pipeline of k_fwd_mfma over steps instead of offsets.
  GRegs g0, g1, g2;
  ARegs a0, a1, a2;
  WRegs w0, w1, w2;
  uint32_t p0 = 0, p1 = 0, p2 = 0;
  const int E = K * nslab;
  At at0{0, 0}, at2, at3;                          // steps e, e + 2, e + 3
  {
    At t{0, 0};
    g_load(t, g0);
    next(t);
    g_load(t, g1);
    next(t);
    g_load(t, g2);
    at2 = at3 = t;
    next(at3);
  }
  {
    At t{0, 0};
    w_load(t, w0);
    next(t);
    w_load(t, w1);
    p0 = a_load(At{0, 0}, g0, a0);
    p1 = a_load(t, g1, a1);
  }
  w_store(0, w0);
  __syncthreads();
  auto step = [&](int e, ARegs& aU, uint32_t& pU, ARegs& aF, uint32_t& pF, GRegs& gU, GRegs& gF,
                  WRegs& wN, WRegs& wF) {
    if (e >= E) return;
    g_load(at3, gU);
    w_load(at2, wF);
    pF = a_load(at2, gF, aF);
    mma(at0, e & 1, aU, pU);
    w_store((e + 1) & 1, wN);
    next(at0);
    next(at2);
    next(at3);
    __syncthreads();
  };
  for (int e = 0; e < E; e += 3) {
    step(e, a0, p0, a2, p2, g0, g2, w1, w2);
    step(e + 1, a1, p1, a0, p0, g1, g0, w2, w0);
    step(e + 2, a2, p2, a1, p1, g2, g1, w0, w1);
  }

  int32_t row;
  if constexpr (PAIRS) {
    row = pair_row(gmap, pt, static_cast<int>(map_row), 0);
  } else {
    if (__any(nonfinite(acc))) {
      sum_over_pairs<TIn, TOut, WT>(gmap, perm, gstride, n_rows, K, x, w, bias, y, C_in, C_out,
                                    tile * TILE_ROWS + uwave * WAVE_ROWS, WAVE_ROWS, col0, COLS,
                                    epi);
      return;
    }
    row = map_row < n_rows ? perm[map_row] : -1;
  }
  store_tile<TIn, TOut, RB, NCB, false, true>(acc, row, bias, y, C_out, col0, lg, epi);
}

template <typename TIn, typename TOut, int WT, int NCH, int NCB, int RB, bool AX, bool AW>
void launch_slab_tile(const Call& c, int C_in, uint32_t w_bytes) {
  constexpr int kTileRows = 4 * RB * 16;
  const int64_t ntiles = view_tiles(c.v, kTileRows);
  const dim3 grid(static_cast<unsigned>(8 * ((ntiles + 7) / 8)),
                  static_cast<unsigned>((c.C_out + NCB * 16 - 1) / (NCB * 16)));
  auto kern = k_fwd_slab<TIn, TOut, NCH, NCB, RB, WT, AX, AW, false>;
  if constexpr (WT != 1)
    if (c.v.pair_off) kern = k_fwd_slab<TIn, TOut, NCH, NCB, RB, WT, AX, AW, true>;
  const ViewArgs a = view_args(c.v);
  kern<<<grid, 256, 0, c.stream>>>(
      a.gmap, a.perm, c.v.gstride, c.v.hdr, a.K, static_cast<const TIn*>(c.x), c.x_bytes,
      static_cast<const TIn*>(c.w), w_bytes, c.bias, static_cast<TOut*>(c.y), C_in, c.C_out,
      ntiles, c.epi);
}

// Rows per tile: 64 when the usual 256 (128 with more than 64 columns) would
// leave compute units without two tiles.  An SC book's n_cap is a loose bound
// where its filter exceeds its stride; its output rows are rarely more than
// its input rows, so those count here.
template <typename TIn, typename TOut, int WT, int NCB>
void launch_slab_cols(const Call& c, int C_in, uint32_t w_bytes) {
  constexpr int RB = NCB <= 4 ? 4 : 2;
  const int64_t rows = c.v.n_src > 0 && c.v.n_src < c.v.n_cap ? c.v.n_src : c.v.n_cap;
  const bool small = rows / (4 * RB * 16) < kSmallLayerTiles;
  if (C_in <= MT<TIn>::KC) {
    if (small)
      launch_slab_tile<TIn, TOut, WT, 1, NCB, 1, true, true>(c, C_in, w_bytes);
    else
      launch_slab_tile<TIn, TOut, WT, 1, NCB, RB, true, true>(c, C_in, w_bytes);
  } else {
    if (small)
      launch_slab_tile<TIn, TOut, WT, 2, NCB, 1, true, true>(c, C_in, w_bytes);
    else
      launch_slab_tile<TIn, TOut, WT, 2, NCB, RB, true, true>(c, C_in, w_bytes);
  }
}

template <typename TIn, typename TOut, int WT>
void launch_slab(const Call& c, int C_in, uint32_t w_bytes) {
  constexpr int EPP = 16 / static_cast<int>(sizeof(TIn));
  // rows of whole 16-byte pieces: x (and W^T) by C_in, W by C_out
  const bool ax = C_in % EPP == 0, aw = WT != 0 || c.C_out % EPP == 0;
  if (ax && aw) {
    // columns per tile: all of them up to 128, else equal shares of at most 128
    const int cb = (c.C_out + 15) / 16, chunks = (cb + 7) / 8, ncb = (cb + chunks - 1) / chunks;
    if (ncb <= 2) launch_slab_cols<TIn, TOut, WT, 2>(c, C_in, w_bytes);
    else if (ncb <= 4) launch_slab_cols<TIn, TOut, WT, 4>(c, C_in, w_bytes);
    else if (ncb <= 6) launch_slab_cols<TIn, TOut, WT, 6>(c, C_in, w_bytes);
    else launch_slab_cols<TIn, TOut, WT, 8>(c, C_in, w_bytes);
    return;
  }
  if constexpr (WT == 0) {
    if (ax) {
      launch_slab_tile<TIn, TOut, WT, 1, 4, 1, true, false>(c, C_in, w_bytes);
      return;
    }
    if (aw) {
      launch_slab_tile<TIn, TOut, WT, 1, 4, 1, false, true>(c, C_in, w_bytes);
      return;
    }
  }
  launch_slab_tile<TIn, TOut, WT, 1, 4, 1, false, WT != 0>(c, C_in, w_bytes);
}

template <typename TIn, typename TOut>
void run_slab(const Call& c, int wmode, int C_in, uint32_t w_bytes) {
  switch (wmode) {
    case 0: launch_slab<TIn, TOut, 0>(c, C_in, w_bytes); break;
    case 1: launch_slab<TIn, TOut, 1>(c, C_in, w_bytes); break;
    default: launch_slab<TIn, TOut, 2>(c, C_in, w_bytes); break;
  }
}

}  // namespace
}  // namespace spc
