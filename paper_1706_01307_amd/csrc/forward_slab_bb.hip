// k_fwd_slab for bf16 inputs and bf16 outputs.
#include "forward_slab.h"

namespace spc {

void forward_slab_bb(const FwdCall& c, int wmode, int C_in, uint32_t w_bytes) {
  run_slab<uint16_t, uint16_t>(c, wmode, C_in, w_bytes);
}

}  // namespace spc
