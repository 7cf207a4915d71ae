// Schedule-3 kernels for bf16 storage, 1 or 2 query tiles (see attn_stitch_impl.h).
#include "attn_stitch_impl.h"

namespace fs {
hipError_t attn_launch_bf16(const AttnArgs& a, int nq, int nk, hipStream_t s) {
  return nq == 1 ? attn_launch_NK<bf16_t, 1>(a, nk, s) : attn_launch_NK<bf16_t, 2>(a, nk, s);
}
}  // namespace fs
