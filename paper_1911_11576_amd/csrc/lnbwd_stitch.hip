// Schedules 1+2 packed (kernel packing + warp composition + block composition, paper
// Section 5.1): LayerNorm backward, hand-written.  The row path (dx: two row reductions,
// broadcast back through registers) and the column path (dgamma, dbeta: reductions over
// all rows, which Section 4.2 lists among the ops with parallelisation needs of their own)
// have no data dependence on each other but share their inputs, so they are packed over the
// same register-resident rows: dy and x are read from HBM exactly once.
//
// Row path: a fixed grid of workgroups walks the rows together (row = step * grid * waves +
// workgroup * waves + wave), one wavefront per row, lane l owns 16-byte vectors l, l+64, ...;
// wave64 all-reduce for sum(g) and sum(g*xhat).  A wavefront requests its rows two steps
// ahead into three register buffers that take turns (none is ever copied): with one wavefront
// per SIMD the time of a step is otherwise the latency of its loads.
// Column path: every lane keeps double-precision running sums for its own columns over all
// rows its wavefront visits (32768-term fp32 sums would not meet a 1e-5 absolute bar).  At
// the end each wavefront writes its sums to an LDS array of its own (the `S` hand-off of
// block composition), the workgroup adds the arrays in wavefront order and writes ONE partial
// row to a plan-owned workspace; a second, small kernel adds the partial rows in a fixed
// order.  No atomics, no tickets, no waiting between workgroups: the hand-off between the two
// kernels is the stream order, and the result is bit-reproducible.
//
// Slot layout (LDS and workspace): slot q*64 + lane with q = r*4K + k*4 + j holds column
// (k*64+lane)*4 + j of reduction r (0 dbeta, 1 dgamma), so that the 64 lanes of one LDS
// instruction touch 64 consecutive doubles (no bank conflicts).  Only the final store of the
// combine kernel maps slots back to columns.
#include <mutex>
#include <set>

#include "dev_common.h"
#include "launchers.h"

namespace fs {

// LDS a workgroup of this schedule may use: one workgroup per CU by design, so nearly all
// of the CU's 160 KB (the volume constraint of shared-memory planning for this schedule)
static constexpr int64_t kLdsMax = 160 * 1024 - 1024;

struct LnBwdArgs {
  const float* dy; const float* x; const float* gamma; const float* mean; const float* rstd;
  float* dx; float* dgamma; float* dbeta;
  int64_t rows; int cols; int nvec; float inv_n;      // nvec: vectors of a row, the last one moved back to end with the row where four do not divide it
  double* part;       // [grid][2*K*256]   one partial row (slot layout) per workgroup
};

// COL: 0 no column outputs, 1 dbeta only (x is not needed), 2 dgamma and dbeta
// EXACT: cols == K*256, no per-vector masking
// PF: row steps requested ahead of the one being worked on
// MAXWG: largest workgroup the instance is launched with (256: one wavefront per SIMD may use the
// whole register file; 512: two share it)
// NT: nontemporal loads, where the rows are of whole vectors
// WHOLE: rows of whole vectors.  Otherwise vectors are read and written at element alignment, through the caches (neighbouring rows share
// lines), and the first elements of a row's last vector, its neighbour's too, count in nothing.
template <int K, bool WANT_DX, int COL, bool EXACT, int PF, int MAXWG, bool WHOLE = true, bool NT = true>
__global__ __launch_bounds__(MAXWG)
void lnbwd_rows_kernel(const LnBwdArgs a) {
  extern __shared__ double lds[];   // [waves][2*K*256] slots
  constexpr bool WANT_COL = COL != 0, NEED_X = WANT_DX || COL == 2;
  constexpr int SLOTS = K * 256;    // per reduction
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  bool vld[K];
  int voff[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int vi = k * 64 + lane;
    vld[k] = EXACT || vi < a.nvec;
    voff[k] = (vld[k] ? vi : 0) * 4;
    if (!WHOLE && vi == a.nvec - 1) voff[k] = a.cols - 4;
  }
  // elements of the lane's last vector that its neighbour holds too (the row's last vector is in the last set)
  const int skip = !WHOLE && (K - 1) * 64 + lane == a.nvec - 1 ? a.nvec * 4 - a.cols : 0;
  auto counts = [&](int k, int j) { return WHOLE || k < K - 1 ? vld[k] : vld[k] && j >= skip; };
  float gam[K][4];
  double dg[K][4], db[K][4];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if constexpr (WANT_DX) Vec<float>::unpack(cached_load<float, WHOLE>(a.gamma + voff[k]), gam[k]);
#pragma unroll
    for (int j = 0; j < 4; ++j) { dg[k][j] = 0.0; db[k][j] = 0.0; }
  }

  asm volatile("" ::: "memory");   // gamma is requested before the rows (the wait below the row requests counts on it)

  // All workgroups advance through the rows together, so at any moment the chip streams one
  // compact window of dy, x and dx, as a one-shot grid would.
  const int64_t row_end = a.rows;
  const int64_t row_step = (int64_t)gridDim.x * waves;
  int64_t row = (int64_t)blockIdx.x * waves + wave;
  // PF + 1 row buffers that take turns: the loop is unrolled PF + 1 times, step p works on buffer p and
  // first requests the row PF steps ahead into the buffer the step before it has finished with.  No buffer is
  // ever copied (a copy of a buffer that was requested only one step ago would wait for it, which is what
  // shifting the buffers down costs), and every request has PF whole steps to arrive.
  constexpr int NB = PF + 1;
  u32x4 rdy[NB][K], rx[NB][K];
  float rmu[NB], rrs[NB];
  auto request = [&](int b, int64_t want) {
    // past the end: row 0, which is in cache by then (no extra HBM traffic); its values are never used (nor, in an
    // update in place, is what its wavefront may be writing there)
    const int64_t r = want < row_end ? want : 0;
    // (loads complete in the order they are issued: the row's mean and rstd, needed first, go first)
    if constexpr (NEED_X) { rmu[b] = a.mean[r]; rrs[b] = a.rstd[r]; }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      auto load = [](const float* p) { return NT ? stream_load<float, WHOLE>(p) : cached_load<float, WHOLE>(p); };
      rdy[b][k] = load(a.dy + r * a.cols + voff[k]);
      if constexpr (NEED_X) rx[b][k] = load(a.x + r * a.cols + voff[k]);
    }
  };
#pragma unroll
  for (int p = 0; p < PF; ++p) request(p, row + p * row_step);
  // gamma has arrived before the row loop starts: a load still pending at its top would put a wait into the
  // loop that, trip after trip, also waits for the rows requested ahead.  Loads complete in the order they
  // were issued, gamma's first: the wait lets the row requests just issued stay in flight (vmcnt = their
  // number; bits 3:0 and 15:14 of the operand, the other counters left alone).
  constexpr int kRowLoads = PF * (K + (NEED_X ? K + 2 : 0));
  static_assert(kRowLoads < 64, "the wait counter has six bits");
  __builtin_amdgcn_s_waitcnt((kRowLoads & 15) | ((kRowLoads >> 4) << 14) | 0x0F70);
  // one step: request the row PF steps ahead, then the arithmetic of row r out of buffer p
  auto step = [&](const int p, const int64_t r) {
    request((p + PF) % NB, r + PF * row_step);
    __builtin_amdgcn_sched_barrier(0);                    // the requests stay ahead of the arithmetic
    float dy[K][4], xv[K][4];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      Vec<float>::unpack(rdy[p][k], dy[k]);
      if constexpr (NEED_X) Vec<float>::unpack(rx[p][k], xv[k]);
    }
    const float rs = NEED_X ? rrs[p] : 0.f, nmurs = NEED_X ? -rmu[p] * rs : 0.f;
    float s1 = 0.f, s2 = 0.f;
    constexpr bool KEEP_G = K * (PF + 1) < 12;
    float g[KEEP_G ? K : 1][4];
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float d = counts(k, j) ? dy[k][j] : 0.f;
        if constexpr (NEED_X) xv[k][j] = fmaf(xv[k][j], rs, nmurs);      // xhat = (x - mu) * rs
        if constexpr (WANT_COL) db[k][j] += (double)d;
        if constexpr (COL == 2) dg[k][j] += (double)(d * xv[k][j]);
        if constexpr (WANT_DX) {
          const float gj = d * gam[k][j];
          if constexpr (KEEP_G) g[k][j] = gj;
          s1 += gj;
          s2 = fmaf(gj, xv[k][j], s2);
        }
      }
    }
    if constexpr (WANT_DX) {
      // dx = (g - c1 - xhat c2) rs, as two fused multiply-adds per element
      const float nc1 = -(group_allreduce<SumOp, 64>(s1) * a.inv_n) * rs;
      const float nc2 = -(group_allreduce<SumOp, 64>(s2) * a.inv_n) * rs;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        float o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          // (with four vectors per lane dy * gamma is multiplied out again rather than kept: sixteen registers
          // fewer is what keeps three row buffers, the fp64 sums and gamma inside the 256 vector registers)
          const float gj = KEEP_G ? g[k][j] : (counts(k, j) ? dy[k][j] : 0.f) * gam[k][j];
          o[j] = fmaf(xv[k][j], nc2, fmaf(gj, rs, nc1));
        }
        if (!WHOLE && k == K - 1 && skip > 0) {
#pragma unroll
          for (int j = 0; j < 4; ++j) if (j >= skip) a.dx[r * a.cols + voff[k] + j] = o[j];
        } else if (vld[k]) {
          stream_store<float, WHOLE>(a.dx + r * a.cols + voff[k], pack16<float>(o));
        }
      }
    }
  };
  // whole trips of PF + 1 steps without a branch inside (one path through the loop: the waits on the
  // requests count exactly), then the last, partial trip
  for (; row + PF * row_step < row_end; row += NB * row_step) {
#pragma unroll
    for (int p = 0; p < NB; ++p) step(p, row + p * row_step);
  }
#pragma unroll
  for (int p = 0; p < NB; ++p)
    if (row + p * row_step < row_end) step(p, row + p * row_step);

  if constexpr (WANT_COL) {
    // ---- block composition: every wavefront's sums into its own LDS array, then the arrays
    // added in wavefront order by all threads, two slots each, straight into the partial row
    constexpr int n2 = 2 * SLOTS;
    double* mine = lds + (int64_t)wave * n2 + lane;
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        mine[(k * 4 + j) * 64] = db[k][j];
        mine[SLOTS + (k * 4 + j) * 64] = dg[k][j];
      }
    __syncthreads();
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    double* out = a.part + (int64_t)blockIdx.x * n2;
    for (int s = threadIdx.x * 2; s < n2; s += blockDim.x * 2) {
      f64x2 t = *reinterpret_cast<const f64x2*>(lds + s);
      for (int w = 1; w < waves; ++w) t += *reinterpret_cast<const f64x2*>(lds + (int64_t)w * n2 + s);
      *reinterpret_cast<f64x2*>(out + s) = t;
    }
  }
}

// Second kernel of the plan: out[col(slot)] = sum over the workgroups' partial rows, in a fixed order
// (256 / SL interleaved slices of partial rows, then the slices in order).  A block owns SL consecutive slots:
// with 16 the 16 lanes of a slice read one whole 128-byte line of a partial row.
template <int SL, int NT = 256>
__global__ __launch_bounds__(NT)
void lnbwd_combine_kernel(const double* __restrict__ part, int groups, int K, int nvec, int cols, float* dgamma, float* dbeta) {
  constexpr int NS = NT / SL;           // slices
  __shared__ double stage[NS][SL + 1];
  const int n2 = 2 * K * 256;
  const int j = threadIdx.x % SL, slice = threadIdx.x / SL;
  const int s = blockIdx.x * SL + j;
  const double* p = part + s;
  const double acc = combine_partials<16, NS>(p, n2, slice, groups, 0.0, [](double a, double b) { return a + b; });
  stage[slice][j] = acc;
  __syncthreads();
  if (slice == 0) {
    double t = stage[0][j];
#pragma unroll
    for (int k = 1; k < NS; ++k) t += stage[k][j];
    // slot -> column
    const int slots = K * 256;
    const int r = s >= slots ? 1 : 0, q = (s - r * slots) >> 6, vi = (q >> 2) * 64 + (s & 63);
    const int col = vi < nvec - 1 ? vi * 4 + (q & 3) : cols - 4 + (q & 3);
    float* o = r ? dgamma : dbeta;
    if (vi < nvec && col >= vi * 4 && o) o[col] = (float)t;
  }
}
constexpr int kCombineSlots = 16;

namespace {

constexpr int kKs[] = {1, 2, 3, 4};
constexpr int kPrefetch = 2;
// Groups up to here load through the caches, with all outputs.  Nontemporally and so, us, from buffers that were in use a pass before and from others:
//   3600 x 1024 14.1, 12.0 and 14.7, 14.8; 4500 x 768 13.4, 11.4 and 13.8, 13.8; 6000 x 512 11.5, 10.6 and 12.0, 12.3; 20000 x 192 12.7, 11.5 and 13.5, 13.8;
//   12000 x 128 10.2, 9.3 and 10.2, 10.3; 2400 x 832 11.2, 11.3 and 12.1, 12.5; 1500 x 1024 10.0, 9.4 and 10.4, 10.7; 1900 x 768 9.0, 8.8 and 9.2, 9.6; 1500 x 256
//   6.6, 6.1 from others
// That is up to 15 % less where the caches hold the rows, and up to 5 % more (below 256 columns up to 9 % less) where they don't.  Beyond, they hold less and less,
// and the line is drawn on the safe side:
// 8768 x 576 15.8, 14.4 and 16.9, 17.2; 6000 x 1000 19.4, 16.8 and 20.2, 19.8; 16384 x 768 29.7, 30.3 and 30.7, 31.9.
constexpr int64_t kCachedBytes = 48ll << 20;

// more than 64 KB of dynamic LDS has to be enabled once per kernel
template <typename Kern>
hipError_t launch_with_lds(Kern kern, const LnBwdArgs& a, int grid, int wg, size_t lds, hipStream_t s) {
  if (lds > 64 * 1024) {
    static std::mutex mu;
    static std::set<const void*> raised;
    std::lock_guard<std::mutex> lock(mu);
    const void* f = reinterpret_cast<const void*>(kern);
    if (!raised.count(f)) {
      const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax);
      if (e != hipSuccess) return e;
      raised.insert(f);
    }
  }
  hipLaunchKernelGGL(kern, dim3(grid), dim3(wg), lds, s, a);
  return hipGetLastError();
}

template <int K, bool EXACT, int MAXWG>
hipError_t launch_KEW(const LnBwdArgs& a, bool want_dx, bool want_col, int grid, int wg, size_t lds,
                      hipStream_t s) {
  const bool need_x_cols = a.dgamma != nullptr;
  if constexpr (MAXWG == 256 || K == 1)
    if (want_dx && want_col && 12 * a.rows * a.cols <= kCachedBytes)
      return launch_with_lds(lnbwd_rows_kernel<K, true, 2, EXACT, kPrefetch, MAXWG, true, false>, a, grid, wg, lds, s);
  if (want_dx && want_col)   // with dx the row is loaded anyway: always the full column path
    return launch_with_lds(lnbwd_rows_kernel<K, true, 2, EXACT, kPrefetch, MAXWG>, a, grid, wg, lds, s);
  if (want_dx) return launch_with_lds(lnbwd_rows_kernel<K, true, 0, EXACT, kPrefetch, MAXWG>, a, grid, wg, 0, s);
  if (need_x_cols) return launch_with_lds(lnbwd_rows_kernel<K, false, 2, EXACT, kPrefetch, MAXWG>, a, grid, wg, lds, s);
  return launch_with_lds(lnbwd_rows_kernel<K, false, 1, EXACT, kPrefetch, MAXWG>, a, grid, wg, lds, s);
}

template <int K>
hipError_t launch_K(const LnBwdArgs& a, bool want_dx, bool want_col, int grid, int wg, size_t lds,
                    hipStream_t s) {
  if (a.cols % 4 != 0) return launch_with_lds(lnbwd_rows_kernel<K, true, 2, false, kPrefetch, 256, false>, a, grid, wg, lds, s);
  const bool exact = a.nvec == K * 64;
  if (wg <= 256) return exact ? launch_KEW<K, true, 256>(a, want_dx, want_col, grid, wg, lds, s)
                              : launch_KEW<K, false, 256>(a, want_dx, want_col, grid, wg, lds, s);
  return exact ? launch_KEW<K, true, 512>(a, want_dx, want_col, grid, wg, lds, s)
               : launch_KEW<K, false, 512>(a, want_dx, want_col, grid, wg, lds, s);
}

}  // namespace

// Rows of no whole number of vectors, with all three outputs.  Replayed graphs, the generated kernel, which is what such rows had (single elements or vectors
// at element alignment, one row ahead), and this one, in us:
//   taken    2000 x 255 11.5 and 6.4, 4407 x 138 8.3 and 7.4, 2000 x 1023 13.9 and 11.1, 20000 x 511 32.3 and 23.9, 10624 x 658 20.0 and 18.9,
//            32768 x 1023 78.8 and 77.8
//   not      from 16385 rows below 160 columns, where 33 to 40 of a wavefront's lanes hold a vector: 32768 x 131 16.1 and 17.9, 32768 x 159 17.6
//            and 17.9 (17000 x 129 13.2 and 11.9)
//   not      below 128 columns, which leave half of the lanes idle and where the partial rows (256 of 4 KB) outweigh the group: 32768 x 127 18.2 and
//            17.9, from cold buffers 20.7 and 21.5; 1100 x 67 0.9 MB, 7.6 and 5.9, 16000 x 99 12.5 and 11.9.  Groups of a few MB would gain by it
// Up to 1024 rows have a launch of their own kind (lnbwd_packed.hip), the fewest the generated kernel.
bool lnbwd_takes_ragged(const LnBwdSpec& sp, const LaunchOpts& opt) {
  return opt.codegen && opt.wg_size == 0 && opt.rows_per_wave == 0 && opt.grid == 0 && sp.cols % 4 != 0 && sp.cols >= 128 && sp.cols <= 1024 && sp.rows > 1024 && (sp.cols >= 160 || sp.rows <= 16384) &&
         sp.out_dx >= 0 && sp.out_dgamma >= 0 && sp.out_dbeta >= 0;
}

bool lnbwd_stitch_plan(const LnBwdSpec& sp, const LaunchOpts& opt, LnBwdLaunch* out, std::string* err) {
  if (sp.cols % 4 != 0 && !lnbwd_takes_ragged(sp, opt)) { *err = "LayerNorm-backward schedule: cols must be a multiple of 4"; return false; }
  // a lane holds its columns' fp64 running sums: 4 vectors of 4 columns is what fits
  if (sp.cols > 1024) { *err = "LayerNorm-backward schedule: cols > 1024 exceed one wavefront's register tile"; return false; }
  LnBwdLaunch l;
  const int need = (int)(((sp.cols + 3) / 4 + 63) / 64);
  l.K = 4;
  for (int k : kKs) if (k >= need) { l.K = k; break; }
  // 4 wavefronts per workgroup and one workgroup per CU: one wavefront per SIMD has the whole
  // register file for its running sums and three row buffers; more wavefronts measured slower
  // ... but for many rows of up to 224 columns, whose steps are too short to hide a row's latency behind.  Four and eight wavefronts, us from buffers in use a
  // pass before (from others):
  //   all outputs  24832 x 128 12.9 and 11.3 (15.3 and 13.1), 50000 x 64 17.7 and 13.9 (21.8 and 16.7), 32768 x 224 19.7 and 19.1, 60000 x 224 31.0 and 30.3
  //   dx alone     20000 x 128 9.0 and 7.3 (9.5 and 8.2), 60000 x 224 27.4 and 26.9 (28.3 and 28.2), 12288 x 224 7.8 and 7.5 (8.3 and 8.4)
  //   column sums  50000 x 128 16.1 and 12.5 (16.8 and 13.5), 60000 x 224 20.6 and 20.1 (21.5 and 21.5), 12288 x 224 8.5 and 8.3 (9.2 and 9.5)
  //   not          9268 x 192 8.4 and 8.6; 32768 x 256 21.0 and 21.3
  // Up to 252 columns with dx and column sums and up to 24576 rows: 12288 x 252 10.5 and 10.3 (12.2 and 12.1), 20000 x 244 14.8 and 14.8; not 60000 x 252 34.2 and
  // 35.7, 60000 x 240 32.2 and 32.5, nor dx alone 20000 x 240 11.4 and 11.3 (12.0 and 12.4), 60000 x 252 30.6 and 32.1, nor sums alone 20000 x 240 10.5 and 10.5 (11.3 and 11.5)
  const bool want_col = sp.out_dgamma >= 0 || sp.out_dbeta >= 0;
  const bool eight = sp.cols % 4 == 0 && sp.rows >= 12288 && (sp.cols <= 224 || (sp.cols < 256 && sp.rows <= 24576 && sp.out_dx >= 0 && want_col));
  l.wg = opt.wg_size ? opt.wg_size : eight ? 512 : 256;
  if (l.wg < 64 || l.wg > 512 || l.wg % 64) { *err = "LayerNorm-backward schedule: wg_size must be a multiple of 64 in [64,512]"; return false; }
  const int waves = l.wg / 64;
  int64_t grid = opt.grid > 0 ? opt.grid : 256;
  const int64_t max_useful = (sp.rows + waves - 1) / waves;
  if (grid > max_useful) grid = max_useful;
  if (grid < 1) grid = 1;
  if (grid > 4096) grid = 4096;
  l.grid = (int)grid;
  l.n_kernels = want_col ? 2 : 1;
  // (a row is read by the one wavefront that writes it, before it does; whole vectors have never taken updates in place)
  l.in_place = sp.cols % 4 != 0;
  l.lds_bytes = want_col ? (int64_t)waves * 2 * l.K * 256 * 8 : 0;
  if (l.lds_bytes > kLdsMax) {
    *err = "LayerNorm-backward schedule: wg_size needs more LDS for the column sums than a CU has";
    return false;
  }
  l.workspace_bytes = want_col ? (int64_t)16 * l.K * 256 * (int64_t)l.grid : 0;
  *out = l;
  return true;
}

std::string lnbwd_stitch_describe(const LnBwdSpec& sp, const LnBwdLaunch& l) {
  char buf[512];
  snprintf(buf, sizeof buf,
           "reduce_s1[GRID-WARP,WARP]; reduce_s2[GRID-WARP,WARP]; dx[GRID-WARP,WARP-THREAD_%d]; "
           "reduce_dgamma[GRID-CTA-THREAD,WARP-THREAD_%d]S; reduce_dbeta[GRID-CTA-THREAD,WARP-THREAD_%d]S "
           "(hand-written kernel; %d partial rows, then a combine kernel%s); cta_num=%d, cta_size=%d",
           l.K * 4, l.K * 4, l.K * 4, l.grid, l.in_place ? "; takes dx in place of dy or x" : "", l.grid, l.wg);
  (void)sp;
  return buf;
}

int lnbwd_stitch_launch(const LnBwdSpec& sp, const LnBwdLaunch& l, const void* const* in, void* const* out,
                        void* workspace, void* stream, std::string* err) {
  if (sp.cols == 0) return 0;
  const bool want_dx = sp.out_dx >= 0;
  const bool want_col = sp.out_dgamma >= 0 || sp.out_dbeta >= 0;
  LnBwdArgs a{};
  a.dy = static_cast<const float*>(in[sp.in_dy]);
  a.x = sp.in_x >= 0 ? static_cast<const float*>(in[sp.in_x]) : nullptr;
  a.gamma = sp.in_gamma >= 0 ? static_cast<const float*>(in[sp.in_gamma]) : nullptr;
  a.mean = sp.in_mean >= 0 ? static_cast<const float*>(in[sp.in_mean]) : nullptr;
  a.rstd = sp.in_rstd >= 0 ? static_cast<const float*>(in[sp.in_rstd]) : nullptr;
  a.dx = want_dx ? static_cast<float*>(out[sp.out_dx]) : nullptr;
  a.dgamma = sp.out_dgamma >= 0 ? static_cast<float*>(out[sp.out_dgamma]) : nullptr;
  a.dbeta = sp.out_dbeta >= 0 ? static_cast<float*>(out[sp.out_dbeta]) : nullptr;
  a.rows = sp.rows; a.cols = (int)sp.cols; a.nvec = (int)((sp.cols + 3) / 4);
  a.inv_n = (float)(1.0 / (double)sp.cols);
  a.part = static_cast<double*>(workspace);
  hipStream_t s = static_cast<hipStream_t>(stream);
  int groups = 0;
  if (sp.rows > 0) {
    if (want_col && !workspace) { *err = "lnbwd_stitch launch: no workspace"; return -1; }
    hipError_t e;
    const size_t lds = (size_t)l.lds_bytes;
    switch (l.K) {
      case 1: e = launch_K<1>(a, want_dx, want_col, l.grid, l.wg, lds, s); break;
      case 2: e = launch_K<2>(a, want_dx, want_col, l.grid, l.wg, lds, s); break;
      case 3: e = launch_K<3>(a, want_dx, want_col, l.grid, l.wg, lds, s); break;
      default: e = launch_K<4>(a, want_dx, want_col, l.grid, l.wg, lds, s); break;
    }
    if (e != hipSuccess) { *err = std::string("lnbwd_stitch launch: ") + hipGetErrorString(e); return -1; }
    groups = l.grid;
  }
  if (want_col) {
    // sums over zero rows are zero: the combine kernel over zero partial rows writes them
    hipLaunchKernelGGL(lnbwd_combine_kernel<kCombineSlots>, dim3(2 * l.K * 256 / kCombineSlots), dim3(256), 0, s, a.part, groups, l.K, a.nvec, a.cols, a.dgamma, a.dbeta);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { *err = std::string("lnbwd_combine launch: ") + hipGetErrorString(e); return -1; }
  }
  return 0;
}

}  // namespace fs
