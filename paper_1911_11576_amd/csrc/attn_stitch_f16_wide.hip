// Schedule-3 kernels for f16 storage, 4 or 8 query tiles (see attn_stitch_impl.h).
#include "attn_stitch_impl.h"

namespace fs {
hipError_t attn_launch_f16_wide(const AttnArgs& a, int nq, int nk, hipStream_t s) {
  return attn_launch_tiles<f16_t, 4, 8>(a, nq, nk, s);
}
}  // namespace fs
