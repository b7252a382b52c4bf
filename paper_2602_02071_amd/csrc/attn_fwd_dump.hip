// The fused attention kernels of attn_fwd.hpp with the score dump of the
// verification entry point.
#include "attn_fwd.hpp"

namespace baps {

hipError_t launch_attention_dump(const AttnParams& p, int D, int block, hipStream_t st)
{
    return launch_any<true>(p, D, block, st);
}

}  // namespace baps
