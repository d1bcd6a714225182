// k_fwd_slab for bf16 inputs and fp32 outputs.
#include "forward_slab.h"

namespace spc {

void forward_slab_bf(const FwdCall& c, int wmode, int C_in, uint32_t w_bytes) {
  run_slab<uint16_t, float>(c, wmode, C_in, w_bytes);
}

}  // namespace spc
