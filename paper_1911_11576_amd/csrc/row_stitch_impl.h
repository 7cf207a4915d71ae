// Schedule 1 (warp composition, paper Section 5.1): an elementwise prologue, one or two
// row reductions whose results are broadcast back to the row, and an elementwise
// epilogue, stitched into one kernel.  A row (or a group of 64/L short rows) lives in
// the VGPRs of one wavefront from its single HBM read to its single HBM write; the
// reductions are wave64 DPP/permlane all-reduces, so the reduced value reaches every
// dependent op through registers and nothing goes through LDS.
//
// Layout: rows are contiguous.  Lane l of a row group owns 16-byte vectors (V elements) l, l+L, ...,
// l+(K-1)L of the row (consecutive lanes read consecutive vectors: fully coalesced).  Where `cols` is not a
// multiple of V (FIT_RAGGED) the row's last vector is moved back to end with the row: its first elements are
// also its neighbour's and count in no reduction; accesses are then aligned to the element only, and the rows of
// a workgroup, one contiguous run of memory, leave through LDS in aligned 16-byte stores.  A wavefront keeps U independent row
// groups in flight per loop iteration; consecutive wavefronts take consecutive row
// groups, so at any moment the chip streams one compact window of the tensors.
//
// This header holds the kernel template and its per-dtype dispatcher; one translation
// unit per storage dtype instantiates it (row_stitch_f32.hip, ...).
#pragma once
#include "dev_common.h"
#include "launchers.h"

namespace fs {

// Unsigned 32-bit division by a launch-time constant as multiply-high, subtract, shifts
// (Granlund & Montgomery's round-up method): q = (t + ((n - t) >> sh1)) >> sh2 with
// t = mulhi(m, n).  Exact for every n < 2^32.
struct FastDiv {
  uint32_t d = 1, m = 1, sh1 = 0, sh2 = 0;
  static FastDiv make(uint32_t d) {
    FastDiv f;
    f.d = d;
    uint32_t l = 0;
    while (l < 32 && ((uint64_t)1 << l) < d) ++l;            // ceil(log2 d)
    f.m = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << l) - d)) / d + 1);
    f.sh1 = l < 1 ? l : 1;
    f.sh2 = l > 0 ? l - 1 : 0;
    return f;
  }
  __device__ __forceinline__ uint32_t div(uint32_t n) const {
    const uint32_t t = __umulhi(m, n);
    return (t + ((n - t) >> sh1)) >> sh2;
  }
};

struct RowArgs {
  const void* x; const void* res; const void* bias; const void* gamma; const void* beta;
  const void* mask; void* y;
  int64_t rows; int cols; int nvec;
  float scale, eps, inv_n;
  float g_mul, g_a0, g_a1;   // gelu: g = g_mul * h / (1 + exp2(h * (g_a0 + g_a1*h*h)))
  FastDiv mask_d1, mask_d2; int64_t ms0, ms1, ms2;
};

// How a row fits the lane tile: exactly (cols == K*L*V: no masking), in whole vectors, or ragged (cols not a
// multiple of V).  The first two of LayerNorm also with gamma and beta requested late (see row_stitch_kernel).
enum RowFit : int { FIT_VECTORS = 0, FIT_EXACT = 1, FIT_RAGGED = 2, FIT_VECTORS_LATE = 3, FIT_EXACT_LATE = 4 };

constexpr float kLog2e = 1.4426950408889634f;

// 1 / sqrt(x) as the hardware's estimate and one Newton step: a correctly rounded square root and division take
// some thirty instructions per row.  The estimate takes a subnormal argument for zero, so one is scaled by 2^24 first
// (eps = 0 and a spread below 1e-19); where the residual is not finite (x = inf, a variance that overflows; x = 0) the
// estimate itself is the answer: 0 or inf.
__device__ __forceinline__ float rsqrt_newton(float x) {
  const bool tiny = x < 0x1p-126f;
  const float s = tiny ? x * 0x1p24f : x;
  const float r = __builtin_amdgcn_rsqf(s);
  const float e = fmaf(-s * r, r, 1.f);
  const float n = e == e ? fmaf(0.5f * r, e, r) : r;
  return tiny ? n * 0x1p12f : n;
}

// VARIANT: 0 LayerNorm, 1 prologue(bias,GELU,residual)+LayerNorm, 2 softmax, 3 softmax with a
// mask of the scores' shape, 4 softmax with a mask broadcast over leading dims
// Bound by HBM, and for 16-bit rows nearly as much by instructions: a lane holds 16 elements and 64 / L rows share a
// reduction's steps, and only the last vector is masked.  From warm buffers (three sets) LayerNorm over 16384 x 1024 bf16 takes
// 13.0 us (13.8 with a row per wavefront, every vector masked and a correctly rounded 1 / sqrt), 16384 x 768 fp32 18.2
// (19.1), 4096 x 512 bf16 3.3 (3.9), but 16384 x 512 bf16 7.8 (7.4); softmax with a key-padding mask over 75648 rows of 197
// fp16 11.4 (46 with one element per access and the row in LDS).
// Whole vectors of the rows are loaded nontemporally at every size.  Ordinary loads are the faster ones only where the same
// buffers were read a pass before (16384 x 1024 bf16 from three sets 11.2 us against 13.0); on buffers new to the pass they
// are slower (13.8 against 13.0; 4096 x 1024 5.3 against 4.3), and behind a kernel that has just written x as well: producer, this kernel
// and a consumer as a graph over new buffers 38.8 us against 36.7, 4096 x 1500 fp32 31.3 against 31.8, 512 x 1024 bf16 8.0 against 7.3.
template <typename T, int VARIANT, int K, int L, int U, int FIT>
__global__ __launch_bounds__(512) void row_stitch_kernel(const RowArgs a) {
  constexpr int V = Vec<T>::V;
  constexpr int G = 64 / L;
  constexpr bool kLN = VARIANT <= 1, kGelu = VARIANT == 1, kMask = VARIANT >= 3, kMaskBcast = VARIANT == 4;
  constexpr bool EXACT = FIT == FIT_EXACT || FIT == FIT_EXACT_LATE, RAGGED = FIT == FIT_RAGGED;
  constexpr bool LATE = kLN && (FIT == FIT_EXACT_LATE || FIT == FIT_VECTORS_LATE);
  const int lane = threadIdx.x & 63;
  const int sub = lane / L, l = lane % L;
  const int waves = blockDim.x >> 6;
  const T* __restrict__ x = static_cast<const T*>(a.x);
  T* __restrict__ y = static_cast<T*>(a.y);

  // K is the least that covers the row, or with 6 and 8 at most one more: only the last vectors can be partial
  constexpr int KFULL = EXACT ? K : K <= 4 ? K - 1 : K - 2;
  bool vld[K];
  int voff[K], dup[K];                 // dup: elements of the vector that the one before it holds too
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int vi = k * L + l;
    vld[k] = k < KFULL || vi < a.nvec;
    voff[k] = (vld[k] ? vi : 0) * V;   // masked-off lanes re-read vector 0: always in bounds
    dup[k] = 0;
    if (RAGGED && k >= KFULL && vi == a.nvec - 1) { dup[k] = a.nvec * V - a.cols; voff[k] = a.cols - V; }
  }
  auto holds = [&](int k) { return k < KFULL || vld[k]; };
  auto counts = [&](int k, int j) { return k < KFULL || (vld[k] && (!RAGGED || j >= dup[k])); };

  // per-column operands (cached loads, kept packed in their storage dtype); an absent
  // operand becomes its neutral element so the per-element code has no conditionals.
  // The bias is needed first and is read up front.  gamma and beta are requested right behind the row, one memory
  // latency for all of them, where wavefronts follow each other on a CU: LayerNorm over 16384 x 1024 fp32 24.6 -> 23.5 us
  // against a request where the epilogue needs them, 16384 x 768 bf16 11.7 -> 10.7.  Where all wavefronts of a launch start at once (LATE), those
  // requests of the first stand before the rows of the last: 4096 x 768 fp32 4.9 us requested late, 5.7 with the row,
  // 4096 x 1024 bf16 4.4 and 5.0.  Nothing is read twice: a one-shot grid visits one row group per wavefront.
  constexpr uint32_t kOne = sizeof(T) == 4 ? 0x3F800000u : (Vec<T>::kOneBits | (Vec<T>::kOneBits << 16));
  u32x4 bia[K];
  if constexpr (kGelu) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      bia[k] = u32x4{0u, 0u, 0u, 0u};
      if (a.bias) bia[k] = cached_load<T, !RAGGED>(static_cast<const T*>(a.bias) + voff[k]);
    }
  }

  const int64_t n_groups = (a.rows + G - 1) / G;
  const int64_t n_iters = (n_groups + U - 1) / U;
  const int wave = threadIdx.x >> 6;
  const int64_t first = (int64_t)blockIdx.x * waves + wave;
  const int64_t stride = (int64_t)gridDim.x * waves;
  extern __shared__ __attribute__((aligned(16))) unsigned char row_stage[];   // RAGGED: the workgroup's rows of y, waves * U * G of them
  T* const stage = reinterpret_cast<T*>(row_stage);

  // all HBM reads of one iteration: the row groups of x and of the second streamed operand
  // (`aux`: the residual, or the mask)
  auto load_groups = [&](int64_t it, u32x4 (&raw)[U][K], u32x4 (&aux)[U][K], int64_t (&row)[U], bool (&rok)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t r = (it * U + u) * G + sub;
      rok[u] = r < a.rows;
      row[u] = rok[u] ? r : a.rows - 1;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        raw[u][k] = stream_load<T, !RAGGED>(x + row[u] * a.cols + voff[k]);
        aux[u][k] = u32x4{0u, 0u, 0u, 0u};
      }
    }
    if constexpr (kGelu) {
      if (a.res) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int k = 0; k < K; ++k)
            aux[u][k] = stream_load<T, !RAGGED>(static_cast<const T*>(a.res) + row[u] * a.cols + voff[k]);
      }
    }
    if constexpr (kMask) {
      const T* __restrict__ mk = static_cast<const T*>(a.mask);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int64_t mrow = row[u];
        if constexpr (kMaskBcast) {
          const uint32_t r32 = (uint32_t)row[u];
          const uint32_t t = a.mask_d2.div(r32), i2 = r32 - t * a.mask_d2.d;
          const uint32_t i0 = a.mask_d1.div(t), i1 = t - i0 * a.mask_d1.d;
          mrow = i0 * a.ms0 + i1 * a.ms1 + i2 * a.ms2;
        }
        // a broadcast mask row is shared by many score rows: cached load; a full mask is touched once: streaming load
#pragma unroll
        for (int k = 0; k < K; ++k)
          aux[u][k] = kMaskBcast ? cached_load<T, !RAGGED>(mk + mrow * a.cols + voff[k]) : stream_load<T, !RAGGED>(mk + mrow * a.cols + voff[k]);
      }
    }
  };

  // (Register double buffering of the next iteration's loads on a persistent grid was tried
  // and measured 10-30% slower than this one-shot form on MI355X.)
  // (A ragged row's loop runs as long as its workgroup has a row, for the barriers: `it` beyond the last
  // group redoes the last row and stores nothing.)
  for (int64_t it = first; (RAGGED ? it - wave : it) < n_iters; it += stride) {
    float v[U][K][V];
    int64_t row[U];
    bool rok[U];
    u32x4 raw[U][K], aux[U][K];
    load_groups(it, raw, aux, row, rok);
    u32x4 gam[kLN ? K : 1], bet[kLN ? K : 1];
    auto load_gamma_beta = [&]() {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        gam[k] = u32x4{kOne, kOne, kOne, kOne};
        bet[k] = u32x4{0u, 0u, 0u, 0u};
        if (a.gamma) gam[k] = cached_load<T, !RAGGED>(static_cast<const T*>(a.gamma) + voff[k]);
        if (a.beta) bet[k] = cached_load<T, !RAGGED>(static_cast<const T*>(a.beta) + voff[k]);
      }
    };
    if constexpr (kLN && !LATE) load_gamma_beta();

    // ---- thread-composed prologue ---------------------------------------------------
    if constexpr (kGelu) {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        float b[V];
        Vec<T>::unpack(bia[k], b);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          float r[V];
          Vec<T>::unpack(raw[u][k], v[u][k]);
          Vec<T>::unpack(aux[u][k], r);
#pragma unroll
          for (int j = 0; j < V; ++j) {
            const float h = v[u][k][j] + b[j];
            // c*h*(1 + tanh(w)) == 2c*h / (1 + exp(-2w)); exp2 overflow gives rcp(inf) = 0
            const float e = __builtin_amdgcn_exp2f(h * (a.g_a0 + a.g_a1 * (h * h)));
            const float g = (a.g_mul * h) * __builtin_amdgcn_rcpf(1.f + e);
            v[u][k][j] = g + r[j];
          }
        }
      }
    } else if constexpr (kMask) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < K; ++k) {
          float mm[V];
          Vec<T>::unpack(raw[u][k], v[u][k]);
          Vec<T>::unpack(aux[u][k], mm);
#pragma unroll
          for (int j = 0; j < V; ++j) v[u][k][j] = v[u][k][j] * a.scale + mm[j];
        }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < K; ++k) {
          Vec<T>::unpack(raw[u][k], v[u][k]);
          if constexpr (VARIANT == 2) {
#pragma unroll
            for (int j = 0; j < V; ++j) v[u][k][j] *= a.scale;
          }
        }
    }

    // one vector of y: to memory, or for ragged rows to the workgroup's tile in LDS
    auto put = [&](int u, int k, int64_t r, bool row_ok, u32x4 w) {
      if constexpr (RAGGED) {
        typedef typename Unaligned16<T>::type W;
        if (vld[k]) *reinterpret_cast<W*>(stage + ((wave * U + u) * G + sub) * a.cols + voff[k]) = (W)w;
      } else if (row_ok && vld[k]) {
        stream_store16(y + r * a.cols + voff[k], w);
      }
    };
    if constexpr (RAGGED) if (it != first) __syncthreads();      // the tile's previous rows have been read

    // ---- row reductions with register broadcast, epilogue, store ---------------------
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (kLN) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
          for (int j = 0; j < V; ++j) s += counts(k, j) ? v[u][k][j] : 0.f;
        const float mean = group_allreduce<SumOp, L>(s) * a.inv_n;
        float q = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
          for (int j = 0; j < V; ++j) {
            v[u][k][j] -= mean;
            q += counts(k, j) ? v[u][k][j] * v[u][k][j] : 0.f;
          }
        if constexpr (LATE) load_gamma_beta();
        const float var = group_allreduce<SumOp, L>(q) * a.inv_n;
        const float rstd = rsqrt_newton(var + a.eps);
#pragma unroll
        for (int k = 0; k < K; ++k) {
          float o[V], gk[V], bk[V];
          Vec<T>::unpack(gam[k], gk);
          Vec<T>::unpack(bet[k], bk);
#pragma unroll
          for (int j = 0; j < V; ++j) o[j] = (v[u][k][j] * rstd) * gk[j] + bk[j];
          put(u, k, row[u], rok[u], pack16<T>(o));
        }
      } else {
        float mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
          for (int j = 0; j < V; ++j) mx = fmaxf(mx, holds(k) ? v[u][k][j] : -INFINITY);
        mx = group_allreduce<MaxOp, L>(mx);
        const float nmx = -mx * kLog2e;
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
          for (int j = 0; j < V; ++j) {
            // exp(z - max) as one fma and one exp2
            const float e = holds(k) ? __builtin_amdgcn_exp2f(fmaf(v[u][k][j], kLog2e, nmx)) : 0.f;
            v[u][k][j] = e;
            s += !RAGGED || counts(k, j) ? e : 0.f;
          }
        s = group_allreduce<SumOp, L>(s);
        const float inv = 1.f / s;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          float o[V];
#pragma unroll
          for (int j = 0; j < V; ++j) o[j] = v[u][k][j] * inv;
          put(u, k, row[u], rok[u], pack16<T>(o));
        }
      }
    }
    if constexpr (RAGGED) {
      // the workgroup's rows as one dense run (it starts on 16 bytes where the rows per workgroup and their
      // length allow, else on 8 or less)
      __syncthreads();
      const int64_t row0 = (it - wave) * U * G;
      const int rows_wg = waves * U * G;
      const int n = (int)(a.rows - row0 < rows_wg ? a.rows - row0 : rows_wg) * a.cols;
      T* o = y + row0 * a.cols;
      for (int i = (int)threadIdx.x * V; i + V <= n; i += (int)blockDim.x * V)
        stream_store<T, false>(o + i, *reinterpret_cast<const u32x4*>(stage + i));
      for (int i = n / V * V + (int)threadIdx.x; i < n; i += (int)blockDim.x) o[i] = stage[i];
    }
  }
}

// ---- per-dtype dispatch over (VARIANT, K, L, U, EXACT) --------------------------------
template <int KV> constexpr int max_rows_in_flight() { return KV <= 8 ? 4 : KV <= 16 ? 2 : 1; }

template <typename T, int VARIANT, int K, int L, int U>
hipError_t row_launch_fit(const RowArgs& a, int fit, int grid, int wg, hipStream_t s) {
  const unsigned lds = fit == FIT_RAGGED ? (unsigned)((wg / 64) * U * (64 / L) * a.cols * (int)sizeof(T)) : 0;
  switch (fit) {
    case FIT_EXACT: hipLaunchKernelGGL((row_stitch_kernel<T, VARIANT, K, L, U, FIT_EXACT>), dim3(grid), dim3(wg), lds, s, a); break;
    case FIT_VECTORS: hipLaunchKernelGGL((row_stitch_kernel<T, VARIANT, K, L, U, FIT_VECTORS>), dim3(grid), dim3(wg), lds, s, a); break;
    case FIT_EXACT_LATE:
      if constexpr (VARIANT <= 1) hipLaunchKernelGGL((row_stitch_kernel<T, VARIANT, K, L, U, FIT_EXACT_LATE>), dim3(grid), dim3(wg), lds, s, a);
      break;
    case FIT_VECTORS_LATE:
      if constexpr (VARIANT <= 1) hipLaunchKernelGGL((row_stitch_kernel<T, VARIANT, K, L, U, FIT_VECTORS_LATE>), dim3(grid), dim3(wg), lds, s, a);
      break;
    default: hipLaunchKernelGGL((row_stitch_kernel<T, VARIANT, K, L, U, FIT_RAGGED>), dim3(grid), dim3(wg), lds, s, a); break;
  }
  return hipGetLastError();
}

template <typename T, int VARIANT, int K, int L>
hipError_t row_launch_U(const RowArgs& a, int U, int fit, int grid, int wg, hipStream_t s) {
  constexpr int kMaxU = max_rows_in_flight<K * Vec<T>::V>();
  if constexpr (kMaxU >= 4) if (U == 4) return row_launch_fit<T, VARIANT, K, L, 4>(a, fit, grid, wg, s);
  if constexpr (kMaxU >= 2) if (U == 2) return row_launch_fit<T, VARIANT, K, L, 2>(a, fit, grid, wg, s);
  return row_launch_fit<T, VARIANT, K, L, 1>(a, fit, grid, wg, s);
}

template <typename T, int VARIANT>
hipError_t row_launch_KL(const RowArgs& a, int K, int L, int U, int fit, int grid, int wg, hipStream_t s) {
  switch (K * 100 + L) {
    case 108: return row_launch_U<T, VARIANT, 1, 8>(a, U, fit, grid, wg, s);
    case 116: return row_launch_U<T, VARIANT, 1, 16>(a, U, fit, grid, wg, s);
    case 364: return row_launch_U<T, VARIANT, 3, 64>(a, U, fit, grid, wg, s);
    case 464: return row_launch_U<T, VARIANT, 4, 64>(a, U, fit, grid, wg, s);
    default: break;
  }
  if constexpr (Vec<T>::V == 4) {
    switch (K * 100 + L) {
      case 132: return row_launch_U<T, VARIANT, 1, 32>(a, U, fit, grid, wg, s);
      case 316: return row_launch_U<T, VARIANT, 3, 16>(a, U, fit, grid, wg, s);
      case 416: return row_launch_U<T, VARIANT, 4, 16>(a, U, fit, grid, wg, s);
      case 332: return row_launch_U<T, VARIANT, 3, 32>(a, U, fit, grid, wg, s);
      case 432: return row_launch_U<T, VARIANT, 4, 32>(a, U, fit, grid, wg, s);
      case 664: return row_launch_U<T, VARIANT, 6, 64>(a, U, fit, grid, wg, s);
      case 864: return row_launch_U<T, VARIANT, 8, 64>(a, U, fit, grid, wg, s);
      default: break;
    }
  } else {
    switch (K * 100 + L) {
      case 216: return row_launch_U<T, VARIANT, 2, 16>(a, U, fit, grid, wg, s);
      case 232: return row_launch_U<T, VARIANT, 2, 32>(a, U, fit, grid, wg, s);
      case 264: return row_launch_U<T, VARIANT, 2, 64>(a, U, fit, grid, wg, s);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t row_launch_dtype(const RowArgs& a, const RowLaunch& rl, hipStream_t s) {
  const bool exact = a.nvec == rl.K * rl.L;
  const int fit = rl.ragged ? FIT_RAGGED : rl.late && rl.variant <= 1 ? (exact ? FIT_EXACT_LATE : FIT_VECTORS_LATE) : exact ? FIT_EXACT : FIT_VECTORS;
  switch (rl.variant) {
    case 0: return row_launch_KL<T, 0>(a, rl.K, rl.L, rl.U, fit, rl.grid, rl.wg, s);
    case 1: return row_launch_KL<T, 1>(a, rl.K, rl.L, rl.U, fit, rl.grid, rl.wg, s);
    case 2: return row_launch_KL<T, 2>(a, rl.K, rl.L, rl.U, fit, rl.grid, rl.wg, s);
    case 3: return row_launch_KL<T, 3>(a, rl.K, rl.L, rl.U, fit, rl.grid, rl.wg, s);
    default: return row_launch_KL<T, 4>(a, rl.K, rl.L, rl.U, fit, rl.grid, rl.wg, s);
  }
}

// defined one per translation unit
hipError_t row_launch_f32(const RowArgs& a, const RowLaunch& rl, hipStream_t s);
hipError_t row_launch_f16(const RowArgs& a, const RowLaunch& rl, hipStream_t s);
hipError_t row_launch_bf16(const RowArgs& a, const RowLaunch& rl, hipStream_t s);

}  // namespace fs
