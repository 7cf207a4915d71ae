// Schedule-3 kernels for bf16 storage, 4 query tiles (see attn_stitch_impl.h).
#include "attn_stitch_impl.h"

namespace fs {
hipError_t attn_launch_bf16_wide(const AttnArgs& a, int nk, hipStream_t s) { return attn_launch_NK<bf16_t, 4>(a, nk, s); }
}  // namespace fs
