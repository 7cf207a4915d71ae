// Schedule 1, wavefront-team form: rows of 2049..32768 elements stay register-resident like in row_stitch, but one row is held by a
// team of W wavefronts (one workgroup).  Wavefront w of the team owns the 1 KB chunks
// w, w+W, w+2W, ... of the row (K chunks per wavefront), so the team reads W consecutive
// kilobytes per step.  Each row reduction is a wave64 all-reduce followed by one exchange
// of W partial values through LDS (block composition for the reduction only; the row
// itself never leaves the registers).
#include "row_stitch_impl.h"

namespace fs {

template <class Op>
__device__ __forceinline__ float team_allreduce(float v, float* slot, int waves, float identity) {
  v = group_allreduce<Op, 64>(v);
  if ((threadIdx.x & 63) == 0) slot[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = identity;
  for (int w = 0; w < waves; ++w) r = Op::apply(r, slot[w]);   // same order in every thread
  return r;
}

template <typename T, int VARIANT, int K, int FIT>
__global__ __launch_bounds__(1024) void row_team_kernel(const RowArgs a) {
  constexpr int V = Vec<T>::V;
  constexpr bool EXACT = FIT == FIT_EXACT, RAGGED = FIT == FIT_RAGGED;
  constexpr int KFULL = EXACT ? K : K <= 4 ? K - 1 : K - 2;    // (as in row_stitch_kernel: only the last chunks can be partial)
  constexpr bool kLN = VARIANT <= 1, kGelu = VARIANT == 1, kMask = VARIANT >= 3, kMaskBcast = VARIANT == 4;
  // two exchange buffers used alternately: a buffer is rewritten only after the barrier of
  // the other reduction has been passed by every wavefront
  __shared__ float exch[2][16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const T* __restrict__ x = static_cast<const T*>(a.x);
  T* __restrict__ y = static_cast<T*>(a.y);
  constexpr uint32_t kOne = sizeof(T) == 4 ? 0x3F800000u : (Vec<T>::kOneBits | (Vec<T>::kOneBits << 16));

  bool vld[K];
  int voff[K], dup[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int vi = (k * waves + w) * 64 + lane;
    vld[k] = k < KFULL || vi < a.nvec;
    voff[k] = (vld[k] ? vi : 0) * V;
    dup[k] = 0;
    if (RAGGED && k >= KFULL && vi == a.nvec - 1) { dup[k] = a.nvec * V - a.cols; voff[k] = a.cols - V; }
  }
  auto counts = [&](int k, int j) { return k < KFULL || (vld[k] && (!RAGGED || j >= dup[k])); };

  for (int64_t row = blockIdx.x; row < a.rows; row += gridDim.x) {
    float v[K][V];
    u32x4 raw[K], aux[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      raw[k] = stream_load<T, !RAGGED>(x + row * a.cols + voff[k]);
      aux[k] = u32x4{0u, 0u, 0u, 0u};
    }
    if constexpr (kGelu) {
      if (a.res) {
#pragma unroll
        for (int k = 0; k < K; ++k) aux[k] = stream_load<T, !RAGGED>(static_cast<const T*>(a.res) + row * a.cols + voff[k]);
      }
    }
    if constexpr (kMask) {
      const T* __restrict__ mk = static_cast<const T*>(a.mask);
      int64_t mrow = row;
      if constexpr (kMaskBcast) {
        const uint32_t r32 = (uint32_t)row;
        const uint32_t t = a.mask_d2.div(r32), i2 = r32 - t * a.mask_d2.d;
        const uint32_t i0 = a.mask_d1.div(t), i1 = t - i0 * a.mask_d1.d;
        mrow = i0 * a.ms0 + i1 * a.ms1 + i2 * a.ms2;
      }
#pragma unroll
      for (int k = 0; k < K; ++k)
        aux[k] = kMaskBcast ? cached_load<T, !RAGGED>(mk + mrow * a.cols + voff[k]) : stream_load<T, !RAGGED>(mk + mrow * a.cols + voff[k]);
    }
    // ---- thread-composed prologue ------------------------------------------------------
#pragma unroll
    for (int k = 0; k < K; ++k) {
      float av[V];
      Vec<T>::unpack(raw[k], v[k]);
      Vec<T>::unpack(aux[k], av);
      if constexpr (kGelu) {
        float b[V];
        u32x4 braw = u32x4{0u, 0u, 0u, 0u};
        if (a.bias) braw = cached_load<T, !RAGGED>(static_cast<const T*>(a.bias) + voff[k]);
        Vec<T>::unpack(braw, b);
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const float h = v[k][j] + b[j];
          const float e = __builtin_amdgcn_exp2f(h * (a.g_a0 + a.g_a1 * (h * h)));
          v[k][j] = (a.g_mul * h) * __builtin_amdgcn_rcpf(1.f + e) + av[j];
        }
      } else if constexpr (kMask) {
#pragma unroll
        for (int j = 0; j < V; ++j) v[k][j] = v[k][j] * a.scale + av[j];
      } else if constexpr (VARIANT == 2) {
#pragma unroll
        for (int j = 0; j < V; ++j) v[k][j] *= a.scale;
      }
    }
    // ---- row reductions across the team, epilogue, store ---------------------------------
    if constexpr (kLN) {
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int j = 0; j < V; ++j) s += counts(k, j) ? v[k][j] : 0.f;
      const float mean = team_allreduce<SumOp>(s, exch[0], waves, 0.f) * a.inv_n;
      float q = 0.f;
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int j = 0; j < V; ++j) {
          v[k][j] -= mean;
          q += counts(k, j) ? v[k][j] * v[k][j] : 0.f;
        }
      const float var = team_allreduce<SumOp>(q, exch[1], waves, 0.f) * a.inv_n;
      const float rstd = rsqrt_newton(var + a.eps);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        u32x4 graw = u32x4{kOne, kOne, kOne, kOne}, braw = u32x4{0u, 0u, 0u, 0u};
        if (a.gamma) graw = cached_load<T, !RAGGED>(static_cast<const T*>(a.gamma) + voff[k]);
        if (a.beta) braw = cached_load<T, !RAGGED>(static_cast<const T*>(a.beta) + voff[k]);
        float o[V], gk[V], bk[V];
        Vec<T>::unpack(graw, gk);
        Vec<T>::unpack(braw, bk);
#pragma unroll
        for (int j = 0; j < V; ++j) o[j] = (v[k][j] * rstd) * gk[j] + bk[j];
        if (vld[k]) stream_store<T, !RAGGED>(y + row * a.cols + voff[k], pack16<T>(o));
      }
    } else {
      float mx = -INFINITY;
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int j = 0; j < V; ++j) mx = fmaxf(mx, vld[k] ? v[k][j] : -INFINITY);
      mx = team_allreduce<MaxOp>(mx, exch[0], waves, -INFINITY);
      const float nmx = -mx * kLog2e;
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const float e = vld[k] ? __builtin_amdgcn_exp2f(fmaf(v[k][j], kLog2e, nmx)) : 0.f;
          v[k][j] = e;
          s += !RAGGED || counts(k, j) ? e : 0.f;
        }
      s = team_allreduce<SumOp>(s, exch[1], waves, 0.f);
      const float inv = 1.f / s;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        float o[V];
#pragma unroll
        for (int j = 0; j < V; ++j) o[j] = v[k][j] * inv;
        if (vld[k]) stream_store<T, !RAGGED>(y + row * a.cols + voff[k], pack16<T>(o));
      }
    }
  }
}

namespace {

template <typename T, int VARIANT, int K>
hipError_t team_launch_fit(const RowArgs& a, int fit, int grid, int wg, hipStream_t s) {
  if (fit == FIT_EXACT) hipLaunchKernelGGL((row_team_kernel<T, VARIANT, K, FIT_EXACT>), dim3(grid), dim3(wg), 0, s, a);
  else if (fit == FIT_VECTORS) hipLaunchKernelGGL((row_team_kernel<T, VARIANT, K, FIT_VECTORS>), dim3(grid), dim3(wg), 0, s, a);
  else hipLaunchKernelGGL((row_team_kernel<T, VARIANT, K, FIT_RAGGED>), dim3(grid), dim3(wg), 0, s, a);
  return hipGetLastError();
}

template <typename T, int VARIANT>
hipError_t team_launch_K(const RowArgs& a, int K, int fit, int grid, int wg, hipStream_t s) {
  switch (K) {
    case 1: return team_launch_fit<T, VARIANT, 1>(a, fit, grid, wg, s);
    case 2: return team_launch_fit<T, VARIANT, 2>(a, fit, grid, wg, s);
    case 3: return team_launch_fit<T, VARIANT, 3>(a, fit, grid, wg, s);
    case 4: return team_launch_fit<T, VARIANT, 4>(a, fit, grid, wg, s);
    default: break;
  }
  if constexpr (Vec<T>::V == 4) {
    if (K == 6) return team_launch_fit<T, VARIANT, 6>(a, fit, grid, wg, s);
    if (K == 8) return team_launch_fit<T, VARIANT, 8>(a, fit, grid, wg, s);
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t team_launch_variant(const RowArgs& a, const RowTeamLaunch& l, hipStream_t s) {
  const int fit = l.ragged ? FIT_RAGGED : a.nvec == l.K * (l.wg / 64) * 64 ? FIT_EXACT : FIT_VECTORS;
  switch (l.variant) {
    case 0: return team_launch_K<T, 0>(a, l.K, fit, l.grid, l.wg, s);
    case 1: return team_launch_K<T, 1>(a, l.K, fit, l.grid, l.wg, s);
    case 2: return team_launch_K<T, 2>(a, l.K, fit, l.grid, l.wg, s);
    case 3: return team_launch_K<T, 3>(a, l.K, fit, l.grid, l.wg, s);
    default: return team_launch_K<T, 4>(a, l.K, fit, l.grid, l.wg, s);
  }
}

int pick_team_K(int need, int kmax) {
  for (int k : {1, 2, 3, 4, 6, 8}) if (k >= need && k <= kmax) return k;
  return -1;
}

}  // namespace

bool row_team_plan(const RowSpec& sp, const LaunchOpts& opt, RowTeamLaunch* out, std::string* err) {
  const int V = 16 / dtype_size(sp.dtype);
  if (sp.cols < V) { *err = "row schedule (team form): row shorter than a 16-byte vector"; return false; }
  if (sp.rows >= (int64_t)1 << 31) { *err = "row schedule: rows >= 2^31"; return false; }
  const int64_t nvec = (sp.cols + V - 1) / V;
  const int kmax = V == 4 ? 8 : 4;       // at most 32 fp32 values of a row per lane
  // smallest team whose lanes hold at most 16 values each, else the smallest that fits at all
  RowTeamLaunch l;
  l.ragged = sp.cols % V != 0;
  int waves = 0;
  if (opt.wg_size) {
    if (opt.wg_size < 128 || opt.wg_size > 1024 || (opt.wg_size & (opt.wg_size - 1))) {
      *err = "row schedule (team form): wg_size must be a power of two in [128,1024]";
      return false;
    }
    waves = opt.wg_size / 64;
  } else {
    for (int wv = 2; wv <= 16 && !waves; wv *= 2)
      if (nvec <= (int64_t)wv * 64 * (16 / V)) waves = wv;
    // ... of any size where that power of two would leave more than three lanes in ten without work:
    // LayerNorm over 4096 rows of 5003 bf16 21.8 -> 16.8 us, of 5000 18.9 -> 17.7, softmax over 4096 of 4099 fp16 16.2 -> 14.2
    // (where it does not, the power of two is the faster one by 1 to 2 %: 2048 x 5120 fp32, 4096 x 6000 bf16; and where whole
    // vectors leave a CU no third team the wider one is: 256 x 5000 bf16 4.0 against 4.2, 600 x 5000 5.1 against 5.0)
    if (waves && (l.ragged || sp.rows > 512)) {
      const int64_t chunks = (nvec + waves * 64 - 1) / (waves * 64);
      if (nvec * 10 < chunks * waves * 64 * 7)
        for (int wv = waves / 2 + 1; wv < waves; ++wv)
          if (nvec <= (int64_t)wv * 64 * (16 / V)) { waves = wv; break; }
    }
    for (int wv = 2; wv <= 16 && !waves; wv *= 2)
      if (nvec <= (int64_t)wv * 64 * kmax) waves = wv;
  }
  if (!waves) { *err = "row schedule (team form): row longer than 16 wavefronts' register tiles (cols > 32768)"; return false; }
  const int need = (int)((nvec + (int64_t)waves * 64 - 1) / ((int64_t)waves * 64));
  l.K = pick_team_K(need, kmax);
  if (l.K < 0) { *err = "row schedule (team form): row does not fit the team's registers"; return false; }
  l.wg = waves * 64;
  int64_t grid = sp.rows;
  if (opt.grid > 0 && opt.grid < grid) grid = opt.grid;
  if (grid > 0x7fffffff) grid = 0x7fffffff;
  l.grid = (int)(grid < 1 ? 1 : grid);
  const bool mask_bcast = !(sp.mask_d1 == 1 && sp.mask_d2 == 1 && sp.mask_stride[0] == 1);
  l.variant = sp.core == CORE_LAYERNORM ? (sp.gelu ? 1 : 0) : (sp.in_mask < 0 ? 2 : mask_bcast ? 4 : 3);
  *out = l;
  return true;
}

std::string row_team_describe(const RowSpec& sp, const RowTeamLaunch& l) {
  char buf[512];
  const char* r1 = sp.core == CORE_LAYERNORM ? "reduce_mean" : "reduce_max";
  const char* r2 = sp.core == CORE_LAYERNORM ? "reduce_var" : "reduce_sum";
  snprintf(buf, sizeof buf, "%s[GRID,CTA]; %s[GRID,CTA]; out[GRID,CTA-THREAD_%d]; cta_num=%d, cta_size=%d", r1, r2,
           l.K * (16 / dtype_size(sp.dtype)), l.grid, l.wg);
  return buf;
}

void row_fill_args(const RowSpec& sp, const void* const* in, void* const* out, RowArgs* a);

int row_team_launch(const RowSpec& sp, const RowTeamLaunch& l, const void* const* in, void* const* out,
                    void* stream, std::string* err) {
  if (sp.rows == 0 || sp.cols == 0) return 0;
  RowArgs a{};
  row_fill_args(sp, in, out, &a);
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e;
  switch (sp.dtype) {
    case DT_F32: e = team_launch_variant<float>(a, l, s); break;
    case DT_F16: e = team_launch_variant<f16_t>(a, l, s); break;
    default: e = team_launch_variant<bf16_t>(a, l, s); break;
  }
  if (e != hipSuccess) { *err = std::string("row_team launch: ") + hipGetErrorString(e); return -1; }
  return 0;
}

}  // namespace fs
