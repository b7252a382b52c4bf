// The fused attention kernels of attn_fwd.hpp as the library's calls run them
// (the score-dump build of the same kernels is a translation unit of its own:
// the two compile side by side).
#include "attn_fwd.hpp"

namespace baps {

hipError_t launch_attention(const AttnParams& p, int D, int block, hipStream_t st)
{
    return p.dump_slot ? launch_attention_dump(p, D, block, st) : launch_any<false>(p, D, block, st);
}

}  // namespace baps
