// Schedule 3 for one query per batch element (a decoding step: a new token against the cached keys and values):
//   s = q K^T -> scale -> (+ additive mask or bias) -> softmax -> P (16-bit) -> o = P V -> (x gate) -> (+ residual),
// optional log-sum-exp.  Both products are matrix-vector products: each of K and V is read once and used once,
// so the kernel is bound by HBM alone, and a matrix-unit tile would do one useful row of sixteen and send K and V
// through LDS to get it.  Instead a wavefront takes a whole batch element with no LDS and no barrier: lane (kl, c) =
// (l / CH, l % CH) reads the 16-byte chunk c of keys kl, kl + 64/CH, ... -- consecutive lanes, consecutive memory --,
// its share of the dot products is summed over the CH lanes of a key, after which those lanes hold the scores
// of just the keys whose V chunks they read: the weights need no exchange either, only the D sums at the end do.
// All K requests of the element are in flight before the first use, V's behind them (or, where the registers do not
// hold both, each in the place of a K chunk that has been used).  The compiler sinks requests towards their uses to
// save registers, which costs a second and a third memory latency: scheduling barriers hold them (HOLD).  From cold buffers,
// bf16: 512 elements x 64 keys x 64 4.9 -> 4.1 us, 128 x 77 x 128 5.5 -> 4.8, 4096 x 33 x 64 8.6 -> 8.0.  Not in the nontemporal form of
// whole tiles without operands and with 32 requests or more per wavefront, where other wavefronts hide what the registers
// cost: 4096 x 128 x 64 22.3 us, 23.2 held.
// Measured, 4096 elements x 128 keys x 64 fp16: 21.5 us, 6.3 TB/s (26.0 on a matrix-unit tile with K and V in LDS);
// 8192 x 128 x 32: 20.5 (38.8); 2048 x 77 x 128 bf16 with a key mask: 14.4 (30.5).
#include "attn_stitch_impl.h"

namespace fs {
namespace {

// the value of the lanes l, l ^ L, l ^ 2L, ... (all that share l % L) summed, in all of them
template <int L> __device__ __forceinline__ float stride_allreduce(float v) {
  if (L <= 4) v += dpp_move<0x124>(v);        // row rotations: by 4, by 8
  if (L <= 8) v += dpp_move<0x128>(v);
  uint32_t u = __builtin_bit_cast(uint32_t, v);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  v = as_f32(r[0]) + as_f32(r[1]);
  u = __builtin_bit_cast(uint32_t, v);
  r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return as_f32(r[0]) + as_f32(r[1]);
}

// NT: 16-key tiles; X: the group has a mask, an epilogue operand or a second output; E: exactly 16 NT keys
template <typename T, int D, int NT, bool X, bool E, bool STREAM>
__global__ __launch_bounds__(256) void attn_decode_kernel(const AttnArgs a) {
  constexpr int CH = D / 8, KPR = 64 / CH, NR = NT * 16 / KPR;      // chunks per key, keys per round of the wavefront, rounds
  constexpr bool BOTH = NR <= 16;                                   // K and V in registers at once
  constexpr bool HOLD = !(STREAM && E && !X && NR >= 16);
  const int lane = threadIdx.x & 63;
  const int b = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
  if (b >= a.batch) return;
  const int kl = lane / CH, c = lane % CH, sk = E ? 16 * NT : a.sk;
  const uint16_t* kb = static_cast<const uint16_t*>(a.k) + (int64_t)b * sk * D + 8 * c;
  const uint16_t* vb = static_cast<const uint16_t*>(a.v) + (int64_t)b * sk * D + 8 * c;
  const int64_t row = (int64_t)b * D + 8 * c;
  auto key_of = [&](int r) { return r * KPR + kl; };
  auto read = [&](const uint16_t* base, int r) {                    // (keys beyond the last: the last again)
    const int key = E ? key_of(r) : min(key_of(r), sk - 1);
    return STREAM ? stream_load16(base + key * D) : *reinterpret_cast<const u32x4*>(base + key * D);
  };
  u32x4 kr[NR], vr[NR];
  const u32x4 qr = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(a.q) + row);
#pragma unroll
  for (int r = 0; r < NR; ++r) kr[r] = read(kb, r);
  float mk[X ? NR : 1];
  u32x4 gt = {0u, 0u, 0u, 0u}, rs = {0u, 0u, 0u, 0u};
  if constexpr (X) {
    if (a.mask) {
      const float* m = a.mask + (int64_t)b * a.mask_sb;
#pragma unroll
      for (int r = 0; r < NR; ++r) mk[r] = m[E ? key_of(r) : min(key_of(r), sk - 1)];
    }
  }
  if constexpr (BOTH) {
#pragma unroll
    for (int r = 0; r < NR; ++r) vr[r] = read(vb, r);
  }
  if constexpr (X) {
    if (a.gate) gt = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(a.gate) + row);
    if (a.res) rs = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(a.res) + row);
  }
  asm volatile("" ::: "memory");     // the requests above stay above
  if constexpr (HOLD) __builtin_amdgcn_sched_barrier(0);

  // ---- scores, in units of log 2, of the keys the lane reads
  constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
  const float sc2 = a.scale * kLog2e;
  float q[8], s[NR], mx = -INFINITY;
  Vec<T>::unpack(qr, q);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    float k[8], t = 0.f;
    Vec<T>::unpack(kr[r], k);
#pragma unroll
    for (int j = 0; j < 8; ++j) t = fmaf(q[j], k[j], t);
    if constexpr (!BOTH) {
      vr[r] = read(vb, r);
      if constexpr (HOLD) __builtin_amdgcn_sched_barrier(0);
    }
    float z = group_allreduce<SumOp, CH>(t) * sc2;
    if constexpr (X) if (a.mask) z = fmaf(mk[r], kLog2e, z);
    if (!E && key_of(r) >= sk) z = -INFINITY;
    s[r] = z;
    mx = fmaxf(mx, z);
  }
  // ---- softmax; every score is held by the CH lanes of its key: a sum over the wavefront counts it CH times
  mx = group_allreduce<MaxOp, 64>(mx);
  float sum = 0.f;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    s[r] = __builtin_amdgcn_exp2f(s[r] - mx);
    sum += s[r];
  }
  sum = group_allreduce<SumOp, 64>(sum) * (1.f / CH);
  const float inv = __builtin_amdgcn_rcpf(sum);
  if constexpr (X) if (a.lse && lane == 0) a.lse[b] = (mx + __builtin_amdgcn_logf(sum)) * kLn2;
  // ---- o = P V, the weights rounded to the dot's dtype
  float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const float p = Mfma<T>::lo(Mfma<T>::pack(s[r] * inv, 0.f));
    const u32x4 raw = E || key_of(r) < sk ? vr[r] : u32x4{0u, 0u, 0u, 0u};
    float v[8];
    Vec<T>::unpack(raw, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = fmaf(p, v[j], o[j]);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = stride_allreduce<CH>(o[j]);
  if constexpr (X) {
    float t[8];
    if (a.gate) {
      Vec<T>::unpack(gt, t);
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] *= t[j];
    }
    if (a.res) {
      Vec<T>::unpack(rs, t);
#pragma unroll
      for (int j = 0; j < 8; ++j) o[j] += t[j];
    }
  }
  if (kl == 0) *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(a.o) + row) = pack16<T>(o);
}

template <typename T, int D, int NT, bool STREAM>
hipError_t decode_launch_form(const AttnArgs& a, int grid, int wg, hipStream_t s) {
  const bool extras = a.mask || a.gate || a.res || a.lse, exact = a.sk == 16 * NT;
  if (extras && exact) hipLaunchKernelGGL((attn_decode_kernel<T, D, NT, true, true, STREAM>), dim3(grid), dim3(wg), 0, s, a);
  else if (extras) hipLaunchKernelGGL((attn_decode_kernel<T, D, NT, true, false, STREAM>), dim3(grid), dim3(wg), 0, s, a);
  else if (exact) hipLaunchKernelGGL((attn_decode_kernel<T, D, NT, false, true, STREAM>), dim3(grid), dim3(wg), 0, s, a);
  else hipLaunchKernelGGL((attn_decode_kernel<T, D, NT, false, false, STREAM>), dim3(grid), dim3(wg), 0, s, a);
  return hipGetLastError();
}

// K and V of up to 12 MB are loaded through the caches.  From warm / cold buffers, ordinary loads against nontemporal ones, bf16: 512
// elements x 64 keys x 64 (8 MB) 2.8 / 4.1 us and 3.6 / 3.6, 512 x 77 x 64 (10 MB) 3.4 / 4.5 and 3.8 / 4.0; 512 x 128 x 64 (17 MB) 4.8 / 5.4
// and 4.7 / 5.0, 1536 x 64 x 64 (25 MB) 6.1 / 6.8 and 5.5 / 6.1.
template <typename T, int D, int NT>
hipError_t decode_launch_one(const AttnArgs& a, int grid, int wg, hipStream_t s) {
  if ((int64_t)a.batch * a.sk * D * 4 > (12ll << 20)) return decode_launch_form<T, D, NT, true>(a, grid, wg, s);
  return decode_launch_form<T, D, NT, false>(a, grid, wg, s);
}

template <typename T, int D>
hipError_t decode_launch_keys(const AttnArgs& a, int grid, int wg, hipStream_t s) {
  switch ((a.sk + 15) / 16) {
    case 1: return decode_launch_one<T, D, 1>(a, grid, wg, s);
    case 2:
      if constexpr (D > 32) return decode_launch_one<T, D, 2>(a, grid, wg, s);      // (of 32: the matrix-unit tile)
      return hipErrorInvalidValue;
    case 3: return decode_launch_one<T, D, 3>(a, grid, wg, s);
    case 4: return decode_launch_one<T, D, 4>(a, grid, wg, s);
    case 5: return decode_launch_one<T, D, 5>(a, grid, wg, s);
    case 6: return decode_launch_one<T, D, 6>(a, grid, wg, s);
    case 7: return decode_launch_one<T, D, 7>(a, grid, wg, s);
    case 8: return decode_launch_one<T, D, 8>(a, grid, wg, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t decode_launch_dim(const AttnArgs& a, int grid, int wg, hipStream_t s) {
  switch (a.dim) {
    case 32: return decode_launch_keys<T, 32>(a, grid, wg, s);
    case 64: return decode_launch_keys<T, 64>(a, grid, wg, s);
    default: return decode_launch_keys<T, 128>(a, grid, wg, s);
  }
}

}  // namespace

hipError_t attn_decode_launch(const AttnArgs& a, bool f16, int grid, int wg, hipStream_t s) {
  return f16 ? decode_launch_dim<f16_t>(a, grid, wg, s) : decode_launch_dim<bf16_t>(a, grid, wg, s);
}

}  // namespace fs
