// Plain streaming copy: the achievable-bandwidth yardstick beside the stitched kernels and
// the calibration kernel for HBM byte counters.  It uses the same access path as the
// stitched kernels (one-shot grid, 16 bytes per lane, nontemporal loads and stores), the
// fastest copy shape measured on MI355X, so that a byte counter reads it the same way.
#include "dev_common.h"
#include "launchers.h"

namespace fs {

__global__ __launch_bounds__(256) void stream_copy_kernel(u32x4* __restrict__ dst,
                                                          const u32x4* __restrict__ src, int64_t nvec) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nvec) stream_store16(dst + i, stream_load16(src + i));
}

int stream_copy_launch(void* dst, const void* src, int64_t bytes, void* stream, std::string* err) {
  const int64_t nvec = bytes / 16;
  if (nvec == 0) return 0;
  const int64_t grid = (nvec + 255) / 256;
  if (grid > 0x7fffffff) { *err = "stream_copy: more than 2^31 workgroups"; return -1; }
  hipLaunchKernelGGL(stream_copy_kernel, dim3((unsigned)grid), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<u32x4*>(dst), static_cast<const u32x4*>(src), nvec);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) { *err = std::string("stream_copy launch: ") + hipGetErrorString(e); return -1; }
  return 0;
}

// Second step of a column reduction whose first step left one double-precision partial row
// per workgroup: out[r][c] = sum over g of partial[r][g][c], summed in a fixed order (64
// interleaved slices, then the slices in order), stored in the output's dtype.
struct ColCombineArgs {
  void* out[8];
  int dtype[8];
  int is_max[8];     // the reduction is a maximum, not a sum
};

// NT threads: a block owns 16 columns of one run of rows (one 128-byte line of every partial row); its
// threads are NT / 16 slices of that run's partial rows.  256 threads for up to 512 partial rows (measured
// 0.8 us faster than 1024 on 256 partial rows of 2048 columns), 1024 beyond, 64 for four and fewer (256 runs of 4 rows of 1024
// values, both kernels of the plan: 28.4 us, with 256 threads 35.3).  MOST rows are requested at a time, see combine_partials; one where
// there is one for a slice at most (sixteen: 36.3 us there), eight from 768 blocks on, which hide the latency by themselves (257 rows of 12000 values and
// two sums 30.3 and 30.8, 16 runs of 1024 x 768 13.9 and 14.2; fewer blocks 226 rows of 520 9.6 and 9.4, 2000 x 3000 18.4 and 18.2).
template <int NT, int MOST>
__global__ __launch_bounds__(NT) void col_combine_kernel(const double* __restrict__ partial, int groups, int64_t total_groups,
                                                         int64_t cols, int64_t stride, const ColCombineArgs args) {
  constexpr int NS = NT / 16;
  __shared__ double part[NS][17];
  const int64_t col_blocks = (cols + 15) / 16;
  const int64_t seg = blockIdx.x / col_blocks;
  const int r = blockIdx.y, j = threadIdx.x & 15, slice = threadIdx.x >> 4;
  const int64_t c = (blockIdx.x % col_blocks) * 16 + j;
  const bool is_max = args.is_max[r] != 0;
  double s = is_max ? -__builtin_inf() : 0.0;
  if (c < cols) {
    const double* p = partial + ((int64_t)r * total_groups + seg * groups) * stride + c;
    s = is_max ? combine_partials<MOST, NS>(p, stride, slice, groups, s, [](double a, double b) { return fmax(a, b); })
               : combine_partials<MOST, NS>(p, stride, slice, groups, s, [](double a, double b) { return a + b; });
  }
  part[slice][j] = s;
  __syncthreads();
  if (slice == 0 && c < cols) {
    double t = part[0][j];
    if (is_max) {
      for (int k = 1; k < NS; ++k) t = fmax(t, part[k][j]);
    } else {
#pragma unroll 8
      for (int k = 1; k < NS; ++k) t += part[k][j];
    }
    void* o = args.out[r];
    const float f = (float)t;
    const int64_t at = seg * cols + c;
    if (args.dtype[r] == DT_F32) static_cast<float*>(o)[at] = f;
    else static_cast<uint16_t*>(o)[at] = (uint16_t)(args.dtype[r] == DT_F16 ? f32_to_f16(f) : f32_to_bf16(f));
  }
}

// partial: [n_red][n_seg * groups][stride, or cols] doubles -- for every reduction and every run of rows, `groups`
// partial rows, added in a fixed order into out[r][n_seg][cols].  n_seg = 1: sums over all rows.
int col_combine_launch(const void* partial, int groups, int64_t cols, int n_red, void* const* out, const int* dtype,
                       void* stream, std::string* err, int64_t n_seg, const int* is_max, int64_t stride) {
  if (n_red <= 0 || cols <= 0 || n_seg <= 0) return 0;
  const int64_t blocks = n_seg * ((cols + 15) / 16);
  if (blocks > 0x7fffffffLL) { *err = "col_combine launch: too many runs of rows for one grid"; return -1; }
  ColCombineArgs a{};
  for (int r = 0; r < n_red && r < 8; ++r) { a.out[r] = out[r]; a.dtype[r] = dtype[r]; a.is_max[r] = is_max ? is_max[r] : 0; }
  const dim3 grid((unsigned)blocks, (unsigned)n_red);
  auto launch = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, static_cast<hipStream_t>(stream), static_cast<const double*>(partial), groups, n_seg * (int64_t)groups, cols,
                       stride ? stride : cols, a);
  };
  if (groups <= 4) launch(col_combine_kernel<64, 1>, 64);
  else if (groups <= 16) launch(col_combine_kernel<256, 1>, 256);
  else if (groups > 512) launch(col_combine_kernel<1024, 16>, 1024);
  else if (blocks * n_red >= 768) launch(col_combine_kernel<256, 8>, 256);
  else launch(col_combine_kernel<256, 16>, 256);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) { *err = std::string("col_combine launch: ") + hipGetErrorString(e); return -1; }
  return 0;
}

}  // namespace fs
