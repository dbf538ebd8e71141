// attn_fwd_stats.hip -- the tiled kernel's instantiations with Eq. 4's row
// statistics (attn_fwd_kernel.h), in a translation unit of their own.
#include "attn_fwd_kernel.h"

namespace sdattn {

hipError_t launch_attn_fwd_tiled_stats(const AttnArgs& a) {
    using Seq = std::make_integer_sequence<int, 32>;   // D = 8, 16, ..., 256
    return a.dtype == kF16 ? dispatch_d<kF16, kStats>(a, Seq{}) : dispatch_d<kBF16, kStats>(a, Seq{});
}

}  // namespace sdattn
