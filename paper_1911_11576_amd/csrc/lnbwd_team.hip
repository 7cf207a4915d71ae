// Schedules 1+2 packed, for rows longer than a wavefront's registers hold (1025 to 4096 columns): LayerNorm backward with T wavefronts to a row.
// As in lnbwd_stitch.hip a fixed grid of workgroups walks the rows together, rows are requested ahead into register buffers that take turns, every lane
// keeps fp64 running sums of its own columns, and a second kernel adds the workgroups' partial rows in a fixed order.  The wavefronts of a row hand each other
// two sums through LDS, behind one barrier a row: the slots take turns with the row buffers.
//
// Any row length: vectors of four elements, the last one of a row moved back to end with the row where four do not divide it (at element alignment then).
//
// An update in place (dx in the buffer of dy or x) is safe: a row is read by the wavefronts that write it, all of it before the barrier that comes before
// the first store.
#include <algorithm>
#include <cstdio>

#include "dev_common.h"
#include "launchers.h"

namespace fs {

namespace {

struct Args {
  const float* dy; const float* x; const float* gamma; const float* mean; const float* rstd;
  float* dx;
  double* part;       // [dgamma, dbeta][workgroups][stride]
  int64_t rows; int cols, nvec, stride; float inv_n;
};

struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

template <bool NT, bool WHOLE> __device__ __forceinline__ u32x4 row_load(const float* p) {
  return NT ? stream_load<float, WHOLE>(p) : cached_load<float, WHOLE>(p);
}

// T wavefronts to a row, K vectors of it in a lane, TEAMS rows to a workgroup at a time, the next ones requested ahead.
// Bound by HBM: 4096 x 4096, 18 or 19 rows to each of 224 workgroups, takes 36.6 us, 48 KB a row at 5.5 TB/s beside the partial rows.
template <int T, int K, int TEAMS, bool WHOLE, bool NT>
__global__ __launch_bounds__(64 * T * TEAMS) void lnbwd_team_kernel(const Args a) {
  constexpr int LANES = 64 * T;
  // Two row buffers that take turns, and with them the exchange slots: one is written again behind another row's barrier only.  (Rows requested two steps
  // ahead, in three buffers, are no faster, us with the second kernel in replayed launches of one plan: 4096 x 4096 44.0 and 44.2, 4587 x 1536 18.8 and 18.8, 1600 x 3502 19.8 and 20.5.)
  constexpr int NB = 2;
  extern __shared__ double lds[];                    // [TEAMS - 1][2 * K * 4][LANES]
  __shared__ float exch[NB][TEAMS][T][2];
  // (the same for a whole wavefront: row addresses are scalar, lanes add 32-bit offsets)
  const int team = TEAMS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / LANES);
  const int lane = threadIdx.x % LANES, wave = (threadIdx.x >> 6) % T;
  int zero = 0;
  asm volatile("" : "+v"(zero));      // keeps the rows' mean and rstd vector loads: scalar ones would be waited for with the LDS exchange
  bool vld[K];
  int col[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int v = k * LANES + lane;
    vld[k] = k < K - 1 || v < a.nvec;
    col[k] = !vld[k] ? 0 : WHOLE || v < a.nvec - 1 ? v * 4 : a.cols - 4;
  }
  // elements of the row's last vector that its neighbour holds too (it is in the last set of vectors)
  const int skip = !WHOLE && (K - 1) * LANES + lane == a.nvec - 1 ? a.nvec * 4 - a.cols : 0;
  // (all sets of vectors but the last are whole)
  auto counts = [&](int k, int j) { return k < K - 1 || (vld[k] && (WHOLE || j >= skip)); };
  float gam[K][4];
  double dg[K][4], db[K][4];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    Vec<float>::unpack(cached_load<float, WHOLE>(a.gamma + col[k]), gam[k]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      dg[k][j] = db[k][j] = 0.0;
    }
  }

  const int64_t row_step = (int64_t)gridDim.x * TEAMS;
  u32x4 rdy[NB][K], rx[NB][K];
  float rmu[NB], rrs[NB];
  auto request = [&](int b, int64_t row0) {
    // past the end: row 0, which is in cache by then; its values are never used (nor, in an update in place, is what is being written there)
    const int64_t want = row0 + team, r = want < a.rows ? want : 0;
    rmu[b] = (a.mean + r)[zero];
    rrs[b] = (a.rstd + r)[zero];
    const float *dy = a.dy + r * a.cols, *x = a.x + r * a.cols;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      rdy[b][k] = row_load<NT, WHOLE>(dy + col[k]);
      rx[b][k] = row_load<NT, WHOLE>(x + col[k]);
    }
  };
  int64_t row0 = (int64_t)blockIdx.x * TEAMS;
  request(0, row0);
  // step p: request the next row, then the arithmetic of row `at` + team out of buffer p; ALL: the row exists for every team
  auto step = [&](auto all_c, const int p, const int64_t at) __attribute__((always_inline)) {
    constexpr bool ALL = decltype(all_c)::value;
    const bool ok = ALL || at + team < a.rows;
    uint32_t there = ok ? ~0u : 0u;
    if (!ALL) asm volatile("" : "+v"(there));             // (a mask, not two ways through the step)
    request((p + 1) % NB, at + row_step);
    __builtin_amdgcn_sched_barrier(0);                    // the requests stay ahead of the arithmetic
    float dy[K][4], xh[K][4];
    const float rs = rrs[p], mu = rmu[p];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      Vec<float>::unpack(rdy[p][k], dy[k]);
      Vec<float>::unpack(rx[p][k], xh[k]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        xh[k][j] = (xh[k][j] - mu) * rs;
        const float g = dy[k][j] * gam[k][j];
        s1 = counts(k, j) ? s1 + g : s1;
        s2 = counts(k, j) ? fmaf(g, xh[k][j], s2) : s2;
        const double d = ALL ? dy[k][j] : as_f32(as_u32(dy[k][j]) & there), h = ALL ? xh[k][j] : as_f32(as_u32(xh[k][j]) & there);
        db[k][j] += d;
        dg[k][j] = fma(d, h, dg[k][j]);
      }
    }
    s1 = group_allreduce<SumOp, 64>(s1);
    s2 = group_allreduce<SumOp, 64>(s2);
    if ((threadIdx.x & 63) == 0) { exch[p][team][wave][0] = s1; exch[p][team][wave][1] = s2; }
    __syncthreads();
    s1 = exch[p][team][0][0]; s2 = exch[p][team][0][1];
#pragma unroll
    for (int t = 1; t < T; ++t) { s1 += exch[p][team][t][0]; s2 += exch[p][team][t][1]; }
    const float c1 = s1 * a.inv_n, c2 = -(s2 * a.inv_n);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      float o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = fmaf(xh[k][j], c2, fmaf(dy[k][j], gam[k][j], -c1)) * rs;
      if (!ALL && !ok) continue;
      float* to = a.dx + (at + team) * a.cols + col[k];      // (a multiply-add instead of dy * gamma kept over the barrier)
      if (!WHOLE && k == K - 1 && skip > 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) if (j >= skip) to[j] = o[j];
      } else if (vld[k]) {
        stream_store<float, WHOLE>(to, pack16<float>(o));
      }
    }
  };
  for (; row0 + row_step + TEAMS <= a.rows; row0 += NB * row_step) {
#pragma unroll
    for (int p = 0; p < NB; ++p) step(Yes{}, p, row0 + p * row_step);
  }
#pragma unroll
  for (int p = 0; p < NB; ++p)
    if (row0 + p * row_step < a.rows) step(No{}, p, row0 + p * row_step);      // (the same for the whole workgroup)

  // the teams' sums, in their order
  if constexpr (TEAMS > 1) {
    if (team > 0) {
      double* mine = lds + (int64_t)(team - 1) * 2 * K * 4 * LANES + lane;
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) { mine[(2 * (k * 4 + j)) * LANES] = dg[k][j]; mine[(2 * (k * 4 + j) + 1) * LANES] = db[k][j]; }
    }
    __syncthreads();
    if (team > 0) return;
#pragma unroll
    for (int t = 1; t < TEAMS; ++t) {
      const double* other = lds + (int64_t)(t - 1) * 2 * K * 4 * LANES + lane;
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) { dg[k][j] += other[(2 * (k * 4 + j)) * LANES]; db[k][j] += other[(2 * (k * 4 + j) + 1) * LANES]; }
    }
  }
  typedef double f64x2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    double* out = a.part + ((int64_t)r * gridDim.x + blockIdx.x) * a.stride;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const auto& s = r ? db[k] : dg[k];
      if (WHOLE) {
        if (!vld[k]) continue;
        *reinterpret_cast<f64x2*>(out + col[k]) = f64x2{s[0], s[1]};
        *reinterpret_cast<f64x2*>(out + col[k] + 2) = f64x2{s[2], s[3]};
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) if (counts(k, j)) out[col[k] + j] = s[j];
      }
    }
  }
}

template <typename Kern>
hipError_t launch_kernel(Kern kern, const Args& a, int grid, int wg, size_t lds, hipStream_t s) {
  hipLaunchKernelGGL(kern, dim3(grid), dim3(wg), lds, s, a);      // (at most 32 KB of LDS)
  return hipGetLastError();
}

// Nontemporal loads: see lnbwd_team_plan.
bool streams(int64_t rows, int64_t cols) { return cols % 4 == 0 && 12 * rows * cols > (160ll << 20); }

template <int T, int K, int TEAMS>
hipError_t launch(const Args& a, int grid, hipStream_t s) {
  const size_t lds = (size_t)(TEAMS - 1) * 2 * K * 4 * 64 * T * 8;
  if (a.cols % 4 != 0) return launch_kernel(lnbwd_team_kernel<T, K, TEAMS, false, false>, a, grid, 64 * T * TEAMS, lds, s);
  if (streams(a.rows, a.cols)) return launch_kernel(lnbwd_team_kernel<T, K, TEAMS, true, true>, a, grid, 64 * T * TEAMS, lds, s);
  return launch_kernel(lnbwd_team_kernel<T, K, TEAMS, true, false>, a, grid, 64 * T * TEAMS, lds, s);
}

}  // namespace

// Doubles from one partial row to the next: whole 128-byte lines, which the second kernel reads (6000 x 3001: 5.9 us without).
static int64_t partial_stride(int64_t cols) { return (cols + 15) / 16 * 16; }

// Launches over three sets of buffers with a plan each, the generated kernel, which is what such rows had (up to 512 workgroups, teams of a power of two of
// wavefronts, ragged rows' buffers copied behind every row), and this one, in us (replayed launches of one plan, whose partial rows share a workspace,
// take up to 8 % longer: 4096 x 4096 45.1 and 44.5).
//   taken       1027 x 1472 12.0 and 10.2, 1500 x 1100 12.8 and 10.7, 3000 x 1280 15.9 and 13.6, 4587 x 1536 23.2 and 18.8, 1326 x 2547 18.7 and 14.9,
//               2564 x 2316 21.9 and 18.1, 5500 x 3072 53.3 and 41.5, 6000 x 3001 56.8 and 44.4, 9000 x 3600 82.9 and 77.3, 4096 x 4096 41.5 and 41.3; 1100 x 4096, where the
//               workspace leaves 128 workgroups, 16.6 and 16.7.  Up to 1024 rows have a launch of their own kind (lnbwd_packed.hip)
//   T           two wavefronts to a row up to 2048 columns, else four, with three or four vectors a lane, four wavefronts to a workgroup: 4 and 2 vectors
//               19.4 for 4587 x 1536, where this is 18.8 (both as 256 workgroups); eight wavefronts to a workgroup 18.9, and 4096 x 4096 48.7 and not 44.0 (one plan)
//   loads       through the caches up to 160 MB: 3000 x 1280 13.6 and nontemporally 15.3 (from cold buffers 15.5 and 15.7), 2564 x 2316 18.0 and 21.7, 3000 x
//               4096 32.2 and 35.6, 4000 x 3072 31.5 and 31.6; beyond, 3500 x 4096 38.5 and 37.2, 10000 x 1536 37.8 and 35.9, 4096 x 4096 43.1 and 41.4, 5500 x
//               3072 41.7 and 39.9, 16000 x 1536 55.6 and 52.5, 7000 x 4096 66.7 and 62.9, but 6000 x 3600 53.1 and 55.3, 9000 x 3600 75.2 and 77.8, and one plan's
//               launches 4096 x 4096 42.7 and 44.5.  Rows at element alignment share lines with their neighbours: always through the caches
//   workgroups  192, of four steps of rows at least (every one of them writes a partial row, all of which are read again): 1027 x 1472 10.1, 256 workgroups
//               11.1; 2564 x 2316 18.7, 128 20.4.  Nontemporally 256: 30000 x 1100 70.5, 224 71.8, 192 76.0 (12000 x 1280 35.9, 35.7 and 36.5, 16000 x 1536 53.2, 52.5
//               and 52.8).  With four wavefronts to a row 224, which no shape loses much by: 192, 224 and 256 take 4096 x 4096 41.5, 41.4 and 41.5, 7000 x 4096
//               63.5, 62.9 and 63.4, 5300 x 4000 49.6, 49.4 and 51.0, 8000 x 2600 50.9, 49.5 and 49.4, 4000 x 3300 37.0, 35.6 and 34.6, 9000 x 3600 80.0, 77.9 and 76.1
//   workspace   within FS_STATIC_SCRATCH_BYTES, which fs_launch_static has, wherever sixteen rows to a workgroup would be
bool lnbwd_team_plan(const LnBwdSpec& sp, const LaunchOpts& opt, LnBwdLaunch* out) {
  if (!opt.codegen || opt.wg_size || opt.rows_per_wave || opt.grid) return false;
  if (sp.out_dx < 0 || sp.out_dgamma < 0 || sp.out_dbeta < 0) return false;
  if (sp.cols <= 1024 || sp.cols > 4096 || sp.rows <= 1024) return false;
  LnBwdLaunch l;
  const int nvec = (int)((sp.cols + 3) / 4);
  l.T = nvec <= 512 ? 2 : 4;
  l.K = (nvec + 64 * l.T - 1) / (64 * l.T);
  l.teams = 4 / l.T;
  l.wg = 256;
  const int64_t few = (sp.rows + 15) / 16, row_bytes = 2 * partial_stride(sp.cols) * 8, cap = FS_STATIC_SCRATCH_BYTES;
  int64_t grid = std::min<int64_t>(!streams(sp.rows, sp.cols) ? 192 : l.T == 2 ? 256 : 224, sp.rows / (4 * l.teams));
  if (grid * row_bytes > cap) grid = std::min(grid, few * 2 * sp.cols * 8 > cap ? std::max(few, cap / row_bytes) : cap / row_bytes);
  l.grid = (int)grid;
  l.n_kernels = 2;
  l.in_place = true;
  l.lds_bytes = (int64_t)(l.teams - 1) * 2 * l.K * 4 * 64 * l.T * 8;
  l.workspace_bytes = row_bytes * l.grid;
  *out = l;
  return true;
}

std::string lnbwd_team_describe(const LnBwdLaunch& l) {
  char buf[512];
  snprintf(buf, sizeof buf,
           "reduce_s1[GRID,WARP_%d]S; reduce_s2[GRID,WARP_%d]S; dx[GRID,WARP_%d-THREAD_%d]; "
           "reduce_dgamma[GRID-CTA-THREAD,WARP_%d-THREAD_%d]S; reduce_dbeta[GRID-CTA-THREAD,WARP_%d-THREAD_%d]S "
           "(hand-written kernel; %d wavefronts to a row, %d partial rows, then a combine kernel; takes dx in place of dy or x); cta_num=%d, cta_size=%d",
           l.T, l.T, l.T, l.K * 4, l.T, l.K * 4, l.T, l.K * 4, l.T, l.grid, l.grid, l.wg);
  return buf;
}

int lnbwd_team_launch(const LnBwdSpec& sp, const LnBwdLaunch& l, const void* const* in, void* const* out, void* workspace, void* stream, std::string* err) {
  if (!workspace) { *err = "lnbwd_team launch: no workspace"; return -1; }
  Args a{};
  a.dy = static_cast<const float*>(in[sp.in_dy]);
  a.x = static_cast<const float*>(in[sp.in_x]);
  a.gamma = static_cast<const float*>(in[sp.in_gamma]);
  a.mean = static_cast<const float*>(in[sp.in_mean]);
  a.rstd = static_cast<const float*>(in[sp.in_rstd]);
  a.dx = static_cast<float*>(out[sp.out_dx]);
  a.part = static_cast<double*>(workspace);
  a.rows = sp.rows; a.cols = (int)sp.cols; a.nvec = (int)((sp.cols + 3) / 4); a.stride = (int)partial_stride(sp.cols);
  a.inv_n = (float)(1.0 / (double)sp.cols);
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e;
  switch (l.T * 8 + l.K) {
    case 2 * 8 + 3: e = launch<2, 3, 2>(a, l.grid, s); break;
    case 2 * 8 + 4: e = launch<2, 4, 2>(a, l.grid, s); break;
    case 4 * 8 + 3: e = launch<4, 3, 1>(a, l.grid, s); break;
    default: e = launch<4, 4, 1>(a, l.grid, s); break;
  }
  if (e != hipSuccess) { *err = std::string("lnbwd_team launch: ") + hipGetErrorString(e); return -1; }
  void* sums[2] = {out[sp.out_dgamma], out[sp.out_dbeta]};
  const int f32[2] = {DT_F32, DT_F32};
  return col_combine_launch(workspace, l.grid, sp.cols, 2, sums, f32, stream, err, 1, nullptr, a.stride);
}

}  // namespace fs
