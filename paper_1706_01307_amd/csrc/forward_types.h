// Types the forward kernels are compiled from: the device header of a rule
// book, the view of a gather map, and a forward call with its epilogue.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace spc {

struct DeviceHeader {          // first bytes of the rule book's allocation
  uint32_t status;             // kSt* bits
  uint32_t pad;
  int64_t n_out;               // output rows (SC: computed on the device)
};

// Forward (forward.hip).  A view names the gather map the output-stationary
// kernels walk: for output position p (rows perm[p], p < hdr->n_out <= n_cap)
// and offset i, gmap[i * gstride + p] = 1 + source row (0: none); n_src rows
// of the source features.
struct FwdView {
  const int32_t* gmap;
  const int32_t* perm;
  int64_t gstride;
  const DeviceHeader* hdr;
  int64_t n_cap;
  int64_t K;
  int64_t K_row;               // offsets one row can have at most
  int64_t n_src;
  // Pair views (K = 1; pair_off not NULL): instead of a map, pair e of offset
  // i < pair_K, pairs[pair_off[i] + e] = (input row, output row), adds row
  // `output row` of the source times W^i to row `input row`, each of which is
  // in one pair; n_cap pairs in all.  gmap, perm and gstride are not read.
  const int32_t* pairs = nullptr;
  const int64_t* pair_off = nullptr;
  int pair_K = 0;
};
// Optional epilogue of a forward.  The networks of Section 5 follow each
// convolution with batch normalisation (at inference a per-channel affine
// map), add the block input back in residual blocks, and apply a ReLU, all at
// the active output sites; fused here into the single store of the output:
//   out[r][n] = act(acc[r][n] * scale[n] + bias[n] + res[r][n])
// scale NULL = 1, res NULL = 0 (res has the output's dtype and layout),
// relu 0 = identity, 1 = max(., 0) with NaN kept.
struct Epilogue {
  const float* scale = nullptr;
  const void* res = nullptr;
  int relu = 0;
};
struct FwdCall {
  FwdView v;
  const void* x;
  uint32_t x_bytes;
  const void* w;
  const float* bias;
  void* y;
  int C_out;
  hipStream_t stream;
  Epilogue epi;
};
void forward_run_w0(const FwdCall& c, int in_dt, int out_dt, int C_in);
void forward_run_w1(const FwdCall& c, int in_dt, int out_dt, int C_in);
void forward_run_w2(const FwdCall& c, int in_dt, int out_dt, int C_in);
// Any channel counts, by the types of inputs and outputs (f: fp32, b: bf16);
// c.x_bytes set, w_bytes the bytes of w (both below 2^31).
void forward_slab_ff(const FwdCall& c, int wmode, int C_in, uint32_t w_bytes);
void forward_slab_fb(const FwdCall& c, int wmode, int C_in, uint32_t w_bytes);
void forward_slab_bf(const FwdCall& c, int wmode, int C_in, uint32_t w_bytes);
void forward_slab_bb(const FwdCall& c, int wmode, int C_in, uint32_t w_bytes);

}  // namespace spc
