// k_fwd_slab for fp32 inputs and fp32 outputs.
#include "forward_slab.h"

namespace spc {

void forward_slab_ff(const FwdCall& c, int wmode, int C_in, uint32_t w_bytes) {
  run_slab<float, float>(c, wmode, C_in, w_bytes);
}

}  // namespace spc
