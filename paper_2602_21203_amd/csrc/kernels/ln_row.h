// The LayerNorm of one row by one wave: reductions, loads and arithmetic shared by the
// LayerNorm kernels and the products that normalise their own input rows (both give the
// same bits).
#pragma once
#include "../common.h"

namespace sq {

typedef float ln_f4v __attribute__((ext_vector_type(4)));


// Cross-lane moves inside 16-lane rows (DPP): quad_perm [1,0,3,2] and [2,3,0,1],
// row_half_mirror, row_mirror.  Each step pairs lane i with a lane of the other
// half of its current group, so after the four steps every lane of a row holds
// the row's combined value (a + b and b + a round alike, so all lanes agree);
// the four row values are then read from lanes 0, 16, 32, 48 and combined as
// (r0 + r1) + (r2 + r3).  No LDS traffic, fixed order, result in every lane.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_read(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_move<0xB1>(v);
  v += dpp_move<0x4E>(v);
  v += dpp_move<0x141>(v);
  v += dpp_move<0x140>(v);
  return (lane_read(v, 0) + lane_read(v, 16)) + (lane_read(v, 32) + lane_read(v, 48));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_move<0xB1>(v));
  v = fmaxf(v, dpp_move<0x4E>(v));
  v = fmaxf(v, dpp_move<0x141>(v));
  v = fmaxf(v, dpp_move<0x140>(v));
  return fmaxf(fmaxf(lane_read(v, 0), lane_read(v, 16)), fmaxf(lane_read(v, 32), lane_read(v, 48)));
}

// Lane j-mapping of a row of H floats: VEC (H a multiple of 256, 16-byte aligned
// rows): element t of the lane is column 256 (t / 4) + 4 lane + t % 4, read and
// written as float4; otherwise column lane + 64 t.  E = elements per lane.
template <int E, bool VEC>
__device__ __forceinline__ int ln_col(int lane, int t) {
  return VEC ? 256 * (t >> 2) + 4 * lane + (t & 3) : lane + 64 * t;
}

template <int E, bool VEC>
__device__ __forceinline__ void ln_load_row(const float* __restrict__ p, int H, int lane, float (&v)[E]) {
  if constexpr (VEC) {
#pragma unroll
    for (int c = 0; c < E / 4; ++c) {
      const ln_f4v x = *reinterpret_cast<const ln_f4v*>(__builtin_assume_aligned(p + 256 * c + 4 * lane, 16));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * c + e] = x[e];
    }
  } else {
#pragma unroll
    for (int t = 0; t < E; ++t) {
      const int j = lane + 64 * t;
      v[t] = j < H ? p[j] : 0.f;
    }
  }
}

// a per-column parameter row (gain, shift) in the lane mapping above, read element by
// element (its start need not be 16-byte aligned); under VEC every column is < H
template <int E, bool VEC>
__device__ __forceinline__ void ln_load_par(const float* __restrict__ p, int H, int lane, float (&v)[E]) {
#pragma unroll
  for (int t = 0; t < E; ++t) {
    const int j = ln_col<E, VEC>(lane, t);
    if constexpr (VEC) v[t] = p[j];
    else v[t] = j < H ? p[j] : 0.f;
  }
}

// x-hat, and act(gain x-hat + shift) (o), of a row in registers; returns 1 / sigma
template <int E, bool VEC>
__device__ __forceinline__ float ln_row(const float (&v)[E], const float (&gv)[E], const float (&bv)[E], int H,
                                        int lane, int act_tanh, float (&xh)[E], float (&o)[E]) {
  float s = 0.f;
#pragma unroll
  for (int t = 0; t < E; ++t) s += v[t];
  const float mean = wave_sum(s) / (float)H;
  float q = 0.f;
#pragma unroll
  for (int t = 0; t < E; ++t) {
    const float dv = ln_col<E, VEC>(lane, t) < H ? v[t] - mean : 0.f;
    q += dv * dv;
  }
  const float var = wave_sum(q) / (float)H;
  const float rs = 1.0f / sqrtf(var + 1e-5f);
#pragma unroll
  for (int t = 0; t < E; ++t) {
    xh[t] = (v[t] - mean) * rs;
    const float a = __builtin_fmaf(gv[t], xh[t], bv[t]);   // the backward recomputes it bit for bit
    o[t] = act_tanh ? tanhf(a) : fmaxf(a, 0.f);
  }
  return rs;
}

}  // namespace sq
