// Schedule-3 kernels for bf16 storage, 8 query tiles (see attn_stitch_impl.h).
#include "attn_stitch_impl.h"

namespace fs {
hipError_t attn_launch_bf16_widest(const AttnArgs& a, int nk, hipStream_t s) { return attn_launch_NK<bf16_t, 8>(a, nk, s); }
}  // namespace fs
