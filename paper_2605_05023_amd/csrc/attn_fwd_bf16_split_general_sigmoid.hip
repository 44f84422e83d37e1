// attn_fwd_bf16_split_general_sigmoid.hip -- general-path bf16 kernels with the
// sigmoid normalisation and the keys split over workgroups.
#include "bf16_kernel.h"

namespace attn {

hipError_t launch_bf16_split_general_sigmoid(const AttnParams& p, int head_dim, hipStream_t stream)
{
    return launch_general_norm<kNormSigmoid, false, true>(p, head_dim, stream);
}

}  // namespace attn
