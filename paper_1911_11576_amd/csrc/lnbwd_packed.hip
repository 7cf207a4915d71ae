// Schedules 1+2 packed in ONE launch: LayerNorm backward of few rows (kernel packing, paper Section 5.1).  The row path
// (dx) and the column path (dgamma, dbeta) share only their inputs, so where these are a few MB each gets workgroups
// of its own and reads them for itself: a workgroup of the row path holds rows in registers, one of the column path goes down all rows of
// a strip of columns.  The second reads come from the caches.  No partial rows, no hand-over, no
// second launch: what the form over many rows (lnbwd_stitch.hip and the generated one) spends on those is most of the time of
// a small group.
//
// An update in place (dx in the buffer of dy or x) is two launches of the same kernel, the strips and behind them the rows, since
// workgroups of one launch would write what others still read.  A row is written by the wavefronts that have all of it in registers.
//
// Any row length: vectors of four elements at element alignment, the last one of a row moved back to end with the row.
#include <cstdio>

#include "dev_common.h"
#include "launchers.h"

namespace fs {

namespace {
constexpr int kThreads = 512;

struct Args {
  const float* dy; const float* x; const float* gamma; const float* mean; const float* rstd;
  float* dx; float* dgamma; float* dbeta;
  int rows, cols, nvec, col_blocks; float inv_n;
};
}  // namespace

// A strip of CB columns: CB / 4 lanes side by side, kThreads / (CB / 4) rows at a time, running sums in double precision.
template <int CB, bool ALIGNED>
static __device__ __forceinline__ void column_strip(const Args& a, int strip) {
  constexpr int LANES = CB / 4, SLOTS = kThreads / LANES, WAVES = kThreads / 64, AHEAD = 8;
  __shared__ double part[WAVES][2][CB];
  const int l = threadIdx.x % LANES, slot = threadIdx.x / LANES;
  const int vec = strip * LANES + l;
  const int col = vec < a.nvec - 1 ? vec * 4 : a.cols - 4;      // (lanes past the last vector redo it and store nothing)
  double dg[4] = {0.0, 0.0, 0.0, 0.0}, db[4] = {0.0, 0.0, 0.0, 0.0};
  for (int r0 = 0; r0 < a.rows; r0 += AHEAD * SLOTS) {
    u32x4 rdy[AHEAD], rx[AHEAD];
    float mu[AHEAD], rs[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      rdy[i] = rx[i] = u32x4{0, 0, 0, 0};
      mu[i] = rs[i] = 0.f;
      if (r0 + i * SLOTS >= a.rows) continue;      // (the same for all lanes)
      const int want = r0 + i * SLOTS + slot, r = want < a.rows ? want : a.rows - 1;
      mu[i] = a.mean[r];
      rs[i] = a.rstd[r];
      rdy[i] = cached_load<float, ALIGNED>(a.dy + (int64_t)r * a.cols + col);
      rx[i] = cached_load<float, ALIGNED>(a.x + (int64_t)r * a.cols + col);
    }
    __builtin_amdgcn_sched_barrier(0);      // all requests before the first use
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      if (r0 + i * SLOTS + slot >= a.rows) continue;
      float d[4], xv[4];
      Vec<float>::unpack(rdy[i], d);
      Vec<float>::unpack(rx[i], xv);
      const float nmurs = -mu[i] * rs[i];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        db[j] += (double)d[j];
        dg[j] += (double)(d[j] * fmaf(xv[j], rs[i], nmurs));
      }
    }
  }
  // the lanes of a wavefront that hold the same columns, then the wavefronts, in a fixed order
#pragma unroll
  for (int m = LANES; m < 64; m <<= 1)
#pragma unroll
    for (int j = 0; j < 4; ++j) { dg[j] += __shfl_xor(dg[j], m); db[j] += __shfl_xor(db[j], m); }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) < LANES) {
#pragma unroll
    for (int j = 0; j < 4; ++j) { part[wave][0][4 * l + j] = dg[j]; part[wave][1][4 * l + j] = db[j]; }
  }
  __syncthreads();
  if (threadIdx.x < 2 * CB) {
    const int which = threadIdx.x / CB, c = threadIdx.x % CB;
    double t = part[0][which][c];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) t += part[w][which][c];
    // column of slot c: the row's last vector holds elements of its neighbour first
    const int v = strip * LANES + c / 4, j = c % 4;
    const int at = v < a.nvec - 1 ? v * 4 + j : a.cols - 4 + j;
    const bool own = v < a.nvec - 1 || (v == a.nvec - 1 && at >= v * 4);
    if (own) (which ? a.dbeta : a.dgamma)[at] = (float)t;
  }
}

// T wavefronts to a row, K vectors of it in a lane.
template <int T, int K, bool ALIGNED>
static __device__ __forceinline__ void rows_of(const Args& a, int block) {
  constexpr int RPW = kThreads / 64 / T;
  __shared__ float exch[RPW][2][T];
  const int lane = threadIdx.x % (64 * T), rl = threadIdx.x / (64 * T);
  const int want = block * RPW + rl;
  const bool ok = want < a.rows;
  const int64_t row = ok ? want : a.rows - 1;
  u32x4 rdy[K], rx[K], rg[K];
  int col[K], skip[K];
  bool vld[K];
  const float mu = a.mean[row], rs = a.rstd[row];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int v = k * 64 * T + lane;
    vld[k] = v < a.nvec;
    col[k] = v < a.nvec - 1 ? v * 4 : a.cols - 4;
    skip[k] = v < a.nvec - 1 ? 0 : a.nvec * 4 - a.cols;      // elements of the last vector that its neighbour holds too
    rdy[k] = cached_load<float, ALIGNED>(a.dy + row * a.cols + col[k]);
    rx[k] = cached_load<float, ALIGNED>(a.x + row * a.cols + col[k]);
    rg[k] = cached_load<float, ALIGNED>(a.gamma + col[k]);
  }
  const float nmurs = -mu * rs;
  float s1 = 0.f, s2 = 0.f, g[K][4], xh[K][4];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    float d[4], gam[4];
    Vec<float>::unpack(rdy[k], d);
    Vec<float>::unpack(rx[k], xh[k]);
    Vec<float>::unpack(rg[k], gam);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      xh[k][j] = fmaf(xh[k][j], rs, nmurs);
      g[k][j] = d[j] * gam[j];
      const bool counted = vld[k] && (ALIGNED || j >= skip[k]);
      s1 = counted ? s1 + g[k][j] : s1;
      s2 = counted ? fmaf(g[k][j], xh[k][j], s2) : s2;
    }
  }
  s1 = group_allreduce<SumOp, 64>(s1);
  s2 = group_allreduce<SumOp, 64>(s2);
  if constexpr (T > 1) {
    const int w = (threadIdx.x >> 6) % T;
    if ((threadIdx.x & 63) == 0) { exch[rl][0][w] = s1; exch[rl][1][w] = s2; }
    __syncthreads();
    s1 = exch[rl][0][0]; s2 = exch[rl][1][0];
#pragma unroll
    for (int t = 1; t < T; ++t) { s1 += exch[rl][0][t]; s2 += exch[rl][1][t]; }
  }
  const float nc1 = -(s1 * a.inv_n) * rs, nc2 = -(s2 * a.inv_n) * rs;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    float o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = fmaf(xh[k][j], nc2, fmaf(g[k][j], rs, nc1));
    if (!ok || !vld[k]) continue;
    float* p = a.dx + row * a.cols + col[k];
    if (ALIGNED || skip[k] == 0) {
      stream_store<float, ALIGNED>(p, pack16<float>(o));
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) if (j >= skip[k]) p[j] = o[j];
    }
  }
}

template <int T, int K, int CB, bool ALIGNED>
__global__ __launch_bounds__(kThreads) void lnbwd_packed_kernel(const Args a) {
  // the strips first: they take longer
  if ((int)blockIdx.x < a.col_blocks) column_strip<CB, ALIGNED>(a, blockIdx.x);
  else rows_of<T, K, ALIGNED>(a, blockIdx.x - a.col_blocks);
}

namespace {
template <int T, int K>
void launch_blocks(const Args& a, int grid, int cb, bool aligned, hipStream_t s) {
  if (cb == 32) {
    if (aligned) hipLaunchKernelGGL((lnbwd_packed_kernel<T, K, 32, true>), dim3(grid), dim3(kThreads), 0, s, a);
    else hipLaunchKernelGGL((lnbwd_packed_kernel<T, K, 32, false>), dim3(grid), dim3(kThreads), 0, s, a);
  } else {
    if (aligned) hipLaunchKernelGGL((lnbwd_packed_kernel<T, K, 16, true>), dim3(grid), dim3(kThreads), 0, s, a);
    else hipLaunchKernelGGL((lnbwd_packed_kernel<T, K, 16, false>), dim3(grid), dim3(kThreads), 0, s, a);
  }
}

template <int T, int K>
void launch(Args a, int grid, int cb, bool aligned, hipStream_t s) {
  if (a.dx == a.dy || a.dx == a.x) {
    launch_blocks<T, K>(a, a.col_blocks, cb, aligned, s);
    grid -= a.col_blocks;
    a.col_blocks = 0;
  }
  launch_blocks<T, K>(a, grid, cb, aligned, s);
}
}  // namespace

// Replayed graphs, the form over many rows and this one, in us.
//   rows     A strip goes down all rows in one workgroup, at some 50 GB/s, so its time grows with them, where the other form pays for partial rows and a
//            second launch.  Up to 1024: 1000 x 1000 11.2 and 8.0, 1000 x 2048 15.1 and 10.7; 1200 x 500 7.1 and 8.4, 1500 x 1280 12.1 and 13.3.  Not
//            below 256, whose plans keep the workspace that callers know them by; it costs those time: 255 x 1024 7.4 and 3.8, 128 x 1024 6.5 and 3.6
//   columns  Up to 4096, what the widest instance holds (two vectors a lane of 512): 800 x 4096 16.0 and 11.7, 256 x 256 5.3 and 3.7
//   strips   32 columns (whole lines) where the rows start on lines or are long or few, else 16: 800 x 1024 6.6 against 7.5 with 16, 800 x 4096 11.7 against
//            15.0, 300 x 1600 4.2 against 4.9; 700 x 1000 7.0 and 6.6, 1000 x 1500 10.8 and 10.0
//   in place (two launches, against the generated kernel) 300 x 1600 12.8 and 7.1, 1000 x 2048 19.8 and 14.8, 700 x 1001 10.9 and 11.0, 1024 x 4096 16.6 and 17.8
bool lnbwd_packed_plan(const LnBwdSpec& sp, const LaunchOpts& opt, LnBwdLaunch* out) {
  if (sp.out_dx < 0 || sp.out_dgamma < 0 || sp.out_dbeta < 0 || opt.wg_size || opt.rows_per_wave || opt.grid) return false;
  if (sp.cols < 4 || sp.cols > 4096 || sp.rows < 256 || sp.rows > 1024) return false;
  LnBwdLaunch l;
  l.packed = true;
  const int nvec = (int)((sp.cols + 3) / 4);
  l.in_place = sp.cols % 4 != 0 || sp.cols > 1024;      // (as of the other form for these rows, the generated one; the hand-written one takes none)
  l.T = nvec <= 256 ? 1 : nvec <= 512 ? 4 : 8;
  l.K = (nvec + 64 * l.T - 1) / (64 * l.T);
  l.strip = sp.cols % 32 == 0 || sp.cols >= 2048 || sp.rows <= 400 ? 32 : 16;
  l.wg = kThreads;
  l.grid = (int)((sp.cols + l.strip - 1) / l.strip + (sp.rows * l.T + 7) / 8);
  l.n_kernels = 1;
  l.lds_bytes = 8 * 2 * l.strip * 8;
  l.workspace_bytes = 0;
  *out = l;
  return true;
}

std::string lnbwd_packed_describe(const LnBwdLaunch& l) {
  char buf[512];
  snprintf(buf, sizeof buf,
           "reduce_s1[GRID,%s]; reduce_s2[GRID,%s]; dx[GRID,%s-THREAD_%d] packed with reduce_dgamma[GRID-CTA,THREAD_4]S; reduce_dbeta[GRID-CTA,THREAD_4]S "
           "(hand-written kernel; a workgroup to a strip of %d columns, the others to rows%s); cta_num=%d, cta_size=%d",
           l.T == 1 ? "WARP" : "CTA", l.T == 1 ? "WARP" : "CTA", l.T == 1 ? "WARP" : "CTA", l.K * 4, l.strip, l.in_place ? "; dx in place of dy or x: the strips first, the rows in a second launch" : "", l.grid, l.wg);
  return buf;
}

int lnbwd_packed_launch(const LnBwdSpec& sp, const LnBwdLaunch& l, const void* const* in, void* const* out, void* stream, std::string* err) {
  Args a{};
  a.dy = static_cast<const float*>(in[sp.in_dy]);
  a.x = static_cast<const float*>(in[sp.in_x]);
  a.gamma = static_cast<const float*>(in[sp.in_gamma]);
  a.mean = static_cast<const float*>(in[sp.in_mean]);
  a.rstd = static_cast<const float*>(in[sp.in_rstd]);
  a.dx = static_cast<float*>(out[sp.out_dx]);
  a.dgamma = static_cast<float*>(out[sp.out_dgamma]);
  a.dbeta = static_cast<float*>(out[sp.out_dbeta]);
  a.rows = (int)sp.rows; a.cols = (int)sp.cols; a.nvec = (int)((sp.cols + 3) / 4);
  a.col_blocks = (int)((sp.cols + l.strip - 1) / l.strip);
  a.inv_n = (float)(1.0 / (double)sp.cols);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool aligned = sp.cols % 4 == 0;
  switch (l.T * 8 + l.K) {
    case 9: launch<1, 1>(a, l.grid, l.strip, aligned, s); break;
    case 10: launch<1, 2>(a, l.grid, l.strip, aligned, s); break;
    case 11: launch<1, 3>(a, l.grid, l.strip, aligned, s); break;
    case 12: launch<1, 4>(a, l.grid, l.strip, aligned, s); break;
    case 34: launch<4, 2>(a, l.grid, l.strip, aligned, s); break;
    default: launch<8, 2>(a, l.grid, l.strip, aligned, s); break;
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) { *err = std::string("lnbwd_packed launch: ") + hipGetErrorString(e); return -1; }
  return 0;
}

}  // namespace fs
