// Schedule-3 kernels for bf16 storage, 1 or 2 query tiles (see attn_stitch_impl.h).
#include "attn_stitch_impl.h"

namespace fs {
hipError_t attn_launch_bf16(const AttnArgs& a, int nq, int nk, hipStream_t s) {
  return attn_launch_tiles<bf16_t, 1, 2>(a, nq, nk, s);
}
}  // namespace fs
