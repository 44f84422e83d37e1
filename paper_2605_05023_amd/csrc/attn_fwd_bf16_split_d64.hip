// attn_fwd_bf16_split_d64.hip -- head-dim-64 instantiations of the
// closed-form-mask softmax kernels with the keys split over workgroups.
#include "bf16_kernel.h"

namespace attn {

hipError_t launch_bf16_split_closed_form_d64(const AttnParams& p, hipStream_t stream)
{
    return launch_closed_form<64, true>(p, stream);
}

}  // namespace attn
