// Host side of schedule 3: geometry, LDS budget, template-notation description and launch (the kernel
// template lives in attn_stitch_impl.h, instantiated per dtype).
#include "attn_stitch_impl.h"

namespace fs {

// LDS budget per workgroup: the volume constraint of shared-memory planning.  72 KB of the
// 160 KB a CU has keeps two workgroups resident (the largest case, 128 keys of 128 values, needs 69 632).
static constexpr int64_t kLdsBudget = 72 * 1024;

static int pow2_tiles(int64_t len) {
  const int need = (int)((len + 15) / 16);
  return need <= 1 ? 1 : need <= 2 ? 2 : need <= 4 ? 4 : 8;
}

bool attn_stitch_plan(const AttnSpec& sp, const LaunchOpts& opt, AttnLaunch* out, int* status, std::string* err) {
  *status = FS_ERR_UNSUPPORTED;
  if (sp.dim != 32 && sp.dim != 64 && sp.dim != 128) { *err = "attention schedule: head dim must be 32, 64 or 128"; return false; }
  if (sp.sq > 128 || sp.sk > 128) { *err = "attention schedule: fine-grained dots only (query and key lengths <= 128)"; return false; }
  if (sp.sk == 0 && sp.sq > 0 && sp.batch > 0) { *err = "attention schedule: softmax over zero keys"; return false; }
  if (sp.batch > 0x7fffffff) { *err = "attention schedule: batch too large"; return false; }
  AttnLaunch l;
  l.nq = pow2_tiles(sp.sq);
  l.nk = pow2_tiles(sp.sk);
  l.wg = 64 * l.nq;
  if (opt.wg_size && opt.wg_size != l.wg) { *err = "attention schedule: wg_size is fixed at 64 per 16 query rows"; *status = FS_ERR_INVALID; return false; }
  l.grid = (int)sp.batch;
  if (sp.sq == 1 && !sp.causal && !(sp.dim == 32 && sp.sk > 8 && sp.sk <= 32)) {
    // one query: matrix-vector products, a wavefront per batch element (attn_decode.hip).  9 to 32 keys of 32 stay on the
    // matrix-unit tile.  Tile and matrix-vector products, bf16 with a key mask, us from warm (cold) buffers: 512 x 16 x 32 2.0 and 2.2 (2.4 and 2.7),
    // 4096 x 16 x 32 2.8 and 2.9 (4.0 and 4.5); the products 4096 x 48 x 32 6.6 and 5.6 (7.3 and 6.4), 4096 x 16 x 64 5.1 and 4.4 (5.7 and 5.3),
    // 4096 x 8 x 128 6.5 and 5.0 (7.6 and 5.7), 512 x 128 x 64 5.4 and 5.0 (6.0 and 5.6).  The tile, as it is now, is level or ahead for up to 8 keys
    // of 32, 12 of 64 and in launches of a few MB too, by 0.5 us at most: 512 x 8 x 32 2.0 and 2.2 (2.4 and 2.7), 4096 x 12 x 64 4.2 and 4.3 (4.8 and
    // 5.3), 512 x 64 x 64 3.1 and 2.8 (4.2 and 4.5).  Up to four wavefronts to a workgroup
    // where that leaves four workgroups for every CU (512 elements of 128 keys of 64 fp16: 5.3 us with one each, 7.0
    // with four on half of the CUs), and one if the caller names the workgroup of a single query tile
    l.decode = true;
    l.wg = opt.wg_size ? opt.wg_size : sp.batch >= 4096 ? 256 : sp.batch >= 2048 ? 128 : 64;
    const int waves = l.wg / 64;
    l.grid = (int)((sp.batch + waves - 1) / waves);
    *out = l;
    *status = FS_OK;
    return true;
  }
  l.lds_bytes = attn_lds_bytes(l.nk, (int)sp.dim);
  if (l.lds_bytes > kLdsBudget) {
    char buf[160];
    snprintf(buf, sizeof buf, "attention schedule: needs %lld bytes of LDS per workgroup, budget is %lld",
             (long long)l.lds_bytes, (long long)kLdsBudget);
    *err = buf;
    *status = FS_ERR_LDS;
    return false;
  }
  *out = l;
  *status = FS_OK;
  return true;
}

std::string attn_stitch_describe(const AttnSpec& sp, const AttnLaunch& l) {
  char buf[640];
  if (l.decode) {
    snprintf(buf, sizeof buf,
             "dot_1[GRID-WARP,WARP]; %ssoftmax[GRID-WARP,WARP]; %sdot_2[GRID-WARP,WARP]; %s%s(one query: matrix-vector products) cta_num=%d, cta_size=%d, lds=0",
             sp.in_mask >= 0 ? "add_mask[GRID-WARP,WARP]; " : "", sp.out_lse >= 0 ? "logsumexp[GRID-WARP,WARP]; " : "",
             sp.in_gate >= 0 ? "multiply_gate[GRID-WARP,WARP-THREAD_8]; " : "", sp.in_res >= 0 ? "add_residual[GRID-WARP,WARP-THREAD_8]; " : "", l.grid, l.wg);
    return buf;
  }
  snprintf(buf, sizeof buf,
           "dot_1[GRID,WARP_16,CTA]; %ssoftmax[GRID,WARP_16,WARP]; %sdot_2[GRID,WARP_16,CTA]S; %s%s"
           "cta_num=%d, cta_size=%d, lds=%lld",
           sp.in_mask >= 0 ? "add_mask[GRID,WARP_16,WARP-THREAD_4]; " : "",
           sp.out_lse >= 0 ? "logsumexp[GRID,WARP_16,WARP]; " : "",
           sp.in_gate >= 0 ? "multiply_gate[GRID,WARP_16,CTA-THREAD_4]; " : "",
           sp.in_res >= 0 ? "add_residual[GRID,WARP_16,CTA-THREAD_4]; " : "",
           l.grid, l.wg, (long long)l.lds_bytes);
  return buf;
}

int attn_stitch_launch(const AttnSpec& sp, const AttnLaunch& l, const void* const* in, void* const* out,
                       void* stream, std::string* err) {
  if (sp.batch == 0 || sp.sq == 0) return 0;
  AttnArgs a{};
  a.q = in[sp.in_q]; a.k = in[sp.in_k]; a.v = in[sp.in_v]; a.o = out[sp.out_o];
  a.mask = sp.in_mask >= 0 ? static_cast<const float*>(in[sp.in_mask]) : nullptr;
  a.mask_sb = sp.mask_sb; a.mask_sq = sp.mask_sq;
  a.mask_vec = (sp.sk % 4 == 0 && sp.mask_sb % 4 == 0 && sp.mask_sq % 4 == 0) ? 1 : 0;
  a.gate = sp.in_gate >= 0 ? in[sp.in_gate] : nullptr;
  a.res = sp.in_res >= 0 ? in[sp.in_res] : nullptr;
  a.lse = sp.out_lse >= 0 ? static_cast<float*>(out[sp.out_lse]) : nullptr;
  a.batch = (int)sp.batch; a.sq = (int)sp.sq; a.sk = (int)sp.sk; a.dim = (int)sp.dim;
  a.scale = sp.scale; a.fill = sp.fill; a.causal = sp.causal ? 1 : 0;
  a.skip_masked_tiles = sp.causal && sp.fill == -INFINITY;
  // Nontemporal stores of O in groups of less than 128 MB, but not in the bare exact form (4096 x 64 x 64 x 64 fp16 from cold
  // buffers 24.5 us with ordinary stores, 25.5 without).  From warm / cold buffers against ordinary stores, 64 wide, bf16: with every
  // operand 512 x 100 x 100 8.8 / 10.5 (9.3 / 11.0), 1536 x 100 x 100 25.0 / 27.5 (27.4 / 28.0), 2500 x 100 x 100 40.3 / 41.0 (40.7 / 41.3); with a key
  // mask only 512 x 100 x 100 7.5 / 8.1 (8.0 / 9.2), 1600 x 128 x 128 21.1 / 24.2 (22.5 / 23.7), 2600 x 128 x 128 34.9 / 35.5 (34.2 / 34.8),
  // 4096 x 128 x 128 51.7 / 52.4 (49.9 / 50.7), 3600 x 64 x 64 22.3 / 24.0 (23.0 / 23.5), 8192 x 64 x 64 49.2 / 50.1 (47.0 / 47.8); with a mask of all scores
  // 512 x 100 x 100 9.9 / 11.5 (10.5 / 12.7), 4096 x 100 x 100 69.4 / 70.9 (70.1 / 71.4); bare 2300 x 100 x 100 23.4 / 25.9 (25.1 / 25.8), 4096 x 100 x 100
  // 41.5 / 42.0 (41.0 / 41.5).  The line is the key mask's and the bare group's; at whole tiles of 64 theirs lies lower (2048 x 64 x 64 12.7 / 15.2 (11.9 /
  // 14.5)).  A kernel that reads O at once finds less of it in the caches: with a consumer, from cold buffers, every operand 512 x 100 x 100 15.7 (15.1),
  // 1536 x 100 x 100 39.2 (38.9), key mask 1600 x 128 x 128 38.0 (35.8).
  a.stream_out = sp.batch * sp.dim * 2 * (sp.sq * (2 + (a.gate != nullptr) + (a.res != nullptr)) + 2 * sp.sk) < (128ll << 20);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool f16 = sp.dtype == DT_F16;
  const hipError_t e = l.decode ? attn_decode_launch(a, f16, l.grid, l.wg, s)
                     : l.nq <= 2 ? (f16 ? attn_launch_f16 : attn_launch_bf16)(a, l.nq, l.nk, s)
                     : l.nq == 4 ? (f16 ? attn_launch_f16_wide : attn_launch_bf16_wide)(a, l.nk, s)
                                 : (f16 ? attn_launch_f16_widest : attn_launch_bf16_widest)(a, l.nk, s);
  if (e != hipSuccess) { *err = std::string("attn_stitch launch: ") + hipGetErrorString(e); return -1; }
  return 0;
}

}  // namespace fs
