// FP32 conv encoder on 32 x 32 inputs (Sec. VI Camera Resolution Analysis: 32 -> 15 ->
// 13 -> 11, 3x3 valid convolutions, the first with stride 2, ReLU after each), one
// image per 1024-thread workgroup, forward and backward each one launch.
//
// The general implicit-GEMM convolutions compute every operand address in index
// arithmetic and take one launch per product; they reached 8 TFLOP/s here.  With an
// image's activations in LDS as channel planes, an operand element's address is a
// per-lane base (its pixel or filter) plus an offset that depends on k alone, read
// from a small LDS table, so v_mfma_f32_16x16x4_f32 (32 cycles) is the bound: 28,000
// matrix-core cycles an image forward, 59,000 backward.  Measured for 250 images
// (one per compute unit) against the general path: forward 26.2 us (90), backward with
// the sum of the partial gradients 58.5 us (478).
//
// Forward: the sums are those of the general convolution, bit for bit (k = (c, tap) in
// slices of 64, four accumulators taking 16 k of a slice each, added in order), so
// that the ReLU masks do not depend on which path ran.  A wave owns 16 pixels x all
// filters.  Backward: per layer, the bias sum, the weight gradient (rows f, columns
// (c, tap), contraction over the output pixels) and the input gradient (over (f, tap)
// of a zero-bordered copy of the gradient, masked by the layer's input); each
// workgroup writes its image's partial gradient, summed in image order afterwards.  An
// output's products are four partial sums here too: the gradients of 250 images are
// 1.8e-7 off their 64-bit values (one accumulator 2.2e-7 and 1.1 us less, the general
// path 2.1e-7).
#include "../common.h"

namespace sq {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kT = 1024, kWaves = kT / 64;

// layer l: CIN x HI x HI -> F x HO x HO
template <int C, int F, int SD, int l> struct Lay {
  static constexpr int O0 = (SD - 3) / 2 + 1;
  static constexpr int CIN = l == 0 ? C : F;
  static constexpr int HI = l == 0 ? SD : O0 - 2 * (l - 1), HO = l == 0 ? O0 : HI - 2, S = l == 0 ? 2 : 1;
  static constexpr int P = HO * HO, PI = HI * HI, K = CIN * 9;
  static constexpr int KR = (K + 3) / 4 * 4 + 1;   // LDS row of a filter: whole steps, odd
  static constexpr int DB = l == 0 ? 0 : 2;        // border of the gradient copy (input gradients read it)
  static constexpr int DS = HO + 2 * DB, DP = DS * DS;
};

__device__ __forceinline__ v4f mfma(float a, float b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// n floats (a multiple of 4, 16-byte aligned) between global memory and LDS
// (and, when dst2 is given, there too)
__device__ __forceinline__ void copy4(const float* __restrict__ src, float* dst, int n, float* dst2 = nullptr) {
  for (int e = 4 * (int)threadIdx.x; e < n; e += 4 * kT) {
    const v4f v = *reinterpret_cast<const v4f*>(src + e);
    *reinterpret_cast<v4f*>(dst + e) = v;
    if (dst2) *reinterpret_cast<v4f*>(dst2 + e) = v;
  }
}
__device__ __forceinline__ void zero4(float* dst, int n) {
  for (int e = 4 * (int)threadIdx.x; e < n; e += 4 * kT) *reinterpret_cast<v4f*>(dst + e) = v4f{0.f, 0.f, 0.f, 0.f};
}

// a layer's weights W[f][K] (flat parameters, any alignment): requested early, then
// stored to LDS rows of KR floats, the steps' padding as zeros
template <class Y, int F> struct Weights {
  static constexpr int N = F * Y::KR, R = (N + kT - 1) / kT;
  float v[R];
  __device__ __forceinline__ void load(const float* __restrict__ W) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int e = (int)threadIdx.x + kT * i, f = e / Y::KR, k = e - f * Y::KR;
      v[i] = f < F && k < Y::K ? W[f * Y::K + k] : 0.f;
    }
  }
  __device__ __forceinline__ void store(float* dst) const {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int e = (int)threadIdx.x + kT * i;
      if (e < N) dst[e] = v[i];
    }
  }
};

// ---------------------------------------------------------------- forward
// offset of k = (c, tap) from a pixel's patch origin
template <class Y> __device__ __forceinline__ void fill_fwd(int* tab) {
  for (int k = threadIdx.x; k < (Y::K + 3) / 4 * 4; k += kT) {
    const int kk = k < Y::K ? k : 0, c = kk / 9, t = kk - 9 * c, ky = t / 3, kx = t - 3 * ky;
    tab[k] = c * Y::PI + ky * Y::HI + kx;
  }
}

// in [CIN][PI], w [F][KR], tab as fill_fwd -> out [F][P], post ReLU (all LDS)
template <class Y, int F>
__device__ __forceinline__ void layer_fwd(const float* in, const float* w, const int* tab,
                                          const float* __restrict__ bias, float* out) {
  constexpr int RT = (Y::P + 15) / 16, CT = F / 16;
  const int lane = threadIdx.x & 63, li = lane & 15, lq = lane >> 4;
  for (int rt = threadIdx.x >> 6; rt < RT; rt += kWaves) {
    const int p = min(16 * rt + li, Y::P - 1), oy = p / Y::HO, ox = p - oy * Y::HO;
    const float* ap = in + oy * Y::S * Y::HI + ox * Y::S;
    const float* bp = w + li * Y::KR + lq;
    v4f acc[4][CT];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int j = 0; j < CT; ++j) acc[a][j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < Y::K; k += 4) {   // lane group lq takes k + lq
      float a = ap[tab[k + lq]];
      if (k + 4 > Y::K) a = k + lq < Y::K ? a : 0.f;
#pragma unroll
      for (int j = 0; j < CT; ++j) acc[(k >> 4) & 3][j] = mfma(a, bp[16 * j * Y::KR + k], acc[(k >> 4) & 3][j]);
    }
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      const int f = 16 * j + li;
      const float bv = bias[f];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = 16 * rt + 4 * lq + q;
        const float v = ((acc[0][j][q] + acc[1][j][q]) + acc[2][j][q]) + acc[3][j][q];
        if (r < Y::P) out[f * Y::P + r] = fmaxf(v + bv, 0.f);
      }
    }
  }
}

struct Ptrs { const float* W[3]; const float* b[3]; };
struct Acts { float* h[3]; };

template <int C, int F, int SD>
__global__ __launch_bounds__(kT) void k_encoder32_fwd(const float* __restrict__ x, Ptrs w, Acts h, float* xsave,
                                                      float* feat2) {
  using L0 = Lay<C, F, SD, 0>;
  using L1 = Lay<C, F, SD, 1>;
  using L2 = Lay<C, F, SD, 2>;
  static_assert(F * L1::P <= C * L0::PI && F * L2::P <= F * L0::P, "activations take the place of dead inputs");
  __shared__ __attribute__((aligned(16))) float ra[C * L0::PI];   // x, then h1
  __shared__ __attribute__((aligned(16))) float rb[F * L0::P];    // h0, then h2
  __shared__ float rw[F * L1::KR];
  __shared__ int tab[L1::K];
  const long long img = blockIdx.x;
  Weights<L0, F> w0;
  Weights<L1, F> w1;
  w0.load(w.W[0]);
  copy4(x + img * C * L0::PI, ra, C * L0::PI, xsave ? xsave + img * C * L0::PI : nullptr);
  w1.load(w.W[1]);
  w0.store(rw);
  fill_fwd<L0>(tab);
  __syncthreads();
  layer_fwd<L0, F>(ra, rw, tab, w.b[0], rb);
  __syncthreads();
  copy4(rb, h.h[0] + img * F * L0::P, F * L0::P);
  w1.store(rw);
  w1.load(w.W[2]);
  fill_fwd<L1>(tab);
  __syncthreads();
  layer_fwd<L1, F>(rb, rw, tab, w.b[1], ra);
  __syncthreads();
  copy4(ra, h.h[1] + img * F * L1::P, F * L1::P);
  w1.store(rw);
  fill_fwd<L2>(tab);
  __syncthreads();
  layer_fwd<L2, F>(ra, rw, tab, w.b[2], rb);
  __syncthreads();
  copy4(rb, h.h[2] + img * F * L2::P, F * L2::P, feat2 ? feat2 + img * F * L2::P : nullptr);
}

// ---------------------------------------------------------------- backward
// k = (f, tap) of an input gradient: {offset in the bordered gradient from an input
// pixel's place, offset of the weights (f, channel 0, tap)}
template <class Y, int F> __device__ __forceinline__ void fill_dx(int2* tab) {
  for (int k = threadIdx.x; k < 9 * F; k += kT) {
    const int f = k / 9, t = k - 9 * f, ky = t / 3, kx = t - 3 * ky;
    tab[k] = make_int2(f * Y::DP - ky * Y::DS - kx, f * Y::KR + t);
  }
}
// output pixel q of a weight gradient: {its place in a gradient plane, its patch origin}
template <class Y> __device__ __forceinline__ void fill_dw(int2* tab) {
  for (int q = threadIdx.x; q < (Y::P + 3) / 4 * 4; q += kT) {
    const int qq = q < Y::P ? q : 0, oy = qq / Y::HO, ox = qq - oy * Y::HO;
    tab[q] = make_int2((oy + Y::DB) * Y::DS + ox + Y::DB, oy * Y::S * Y::HI + ox * Y::S);
  }
}

// The steps of a contraction over K as the general convolutions (and the forward) order
// them: slices of 64, four accumulators taking 16 k of a slice each; step(k, accumulator)
// for every whole step of 4.
template <int K, class STEP> __device__ __forceinline__ void slices(const STEP& step) {
#pragma unroll 1
  for (int s = 0; s < K / 64 * 64; s += 64)
#pragma unroll
    for (int i = 0; i < 64; i += 4) step(s + i, i >> 4);
#pragma unroll
  for (int k = K / 64 * 64; k < K / 4 * 4; k += 4) step(k, (k >> 4) & 3);
}
__device__ __forceinline__ v4f sum4(v4f a, v4f b, v4f c, v4f d) { return ((a + b) + c) + d; }

// 16 input pixels x all channels of layer Y's input gradient from D [F][DP], masked by
// the layer's input hin [CIN][PI] > 0, into the interior of the layer below's gradient
// (Z: that layer) [CIN][Z::DP]
template <class Y, class Z, int F>
__device__ __forceinline__ void dx_task(int rt, const float* D, const float* w, const int2* tab, const float* hin,
                                        float* Dn) {
  constexpr int CT = Y::CIN / 16;
  const int lane = threadIdx.x & 63, li = lane & 15, lq = lane >> 4;
  const int p = min(16 * rt + li, Y::PI - 1), iy = p / Y::HI, ix = p - iy * Y::HI;
  const float* ap = D + (iy + 2) * Y::DS + ix + 2;
  const float* bp = w + 9 * li;
  v4f acc[4][CT];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[s][j] = v4f{0.f, 0.f, 0.f, 0.f};
  static_assert(9 * F % 4 == 0, "whole steps");
  slices<9 * F>([&](int k, int s) {
    const int2 o = tab[k + lq];
    const float a = ap[o.x];
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[s][j] = mfma(a, bp[o.y + 144 * j], acc[s][j]);
  });
#pragma unroll
  for (int j = 0; j < CT; ++j) {
    const int c = 16 * j + li;
    const v4f sum = sum4(acc[0][j], acc[1][j], acc[2][j], acc[3][j]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 16 * rt + 4 * lq + q;
      if (r >= Y::PI) continue;
      const int yy = r / Y::HI, xx = r - yy * Y::HI;
      Dn[c * Z::DP + (yy + Z::DB) * Z::DS + xx + Z::DB] = hin[c * Y::PI + r] > 0.f ? sum[q] : 0.f;
    }
  }
}

// columns (c, tap) 16 t .. 16 t + 15 of layer Y's weight gradient, all filters
template <class Y, int F>
__device__ __forceinline__ void dw_task(int t, const float* D, const float* in, const int2* tab,
                                        float* __restrict__ partW) {
  constexpr int RT = F / 16;
  const int lane = threadIdx.x & 63, li = lane & 15, lq = lane >> 4;
  const int kc = min(16 * t + li, Y::K - 1), c = kc / 9, tap = kc - 9 * c, ky = tap / 3, kx = tap - 3 * ky;
  const float* ap = D + li * Y::DP;
  const float* bp = in + c * Y::PI + ky * Y::HI + kx;
  v4f acc[4][RT];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < RT; ++j) acc[s][j] = v4f{0.f, 0.f, 0.f, 0.f};
  slices<Y::P>([&](int q, int s) {
    const int2 o = tab[q + lq];
    const float b = bp[o.y];
#pragma unroll
    for (int j = 0; j < RT; ++j) acc[s][j] = mfma(ap[16 * j * Y::DP + o.x], b, acc[s][j]);
  });
  if constexpr (Y::P % 4 != 0) {   // the last pixels: zeros past the end
    constexpr int q = Y::P / 4 * 4, s = (q >> 4) & 3;
    const int2 o = tab[q + lq];
    const bool ok = q + lq < Y::P;
    const float b = ok ? bp[o.y] : 0.f;
#pragma unroll
    for (int j = 0; j < RT; ++j) acc[s][j] = mfma(ok ? ap[16 * j * Y::DP + o.x] : 0.f, b, acc[s][j]);
  }
  if (16 * t + li < Y::K) {
#pragma unroll
    for (int j = 0; j < RT; ++j) {
      const v4f sum = sum4(acc[0][j], acc[1][j], acc[2][j], acc[3][j]);
#pragma unroll
      for (int q = 0; q < 4; ++q) partW[(16 * j + 4 * lq + q) * Y::K + kc] = sum[q];
    }
  }
}

// bias gradients: a wave sums a filter's plane (its border is zero)
template <class Y, int F>
__device__ __forceinline__ void db_sums(const float* D, float* __restrict__ partb) {
  const int lane = threadIdx.x & 63;
  for (int f = threadIdx.x >> 6; f < F; f += kWaves) {
    float s = 0.f;
    for (int p = lane; p < Y::DP; p += 64) s += D[f * Y::DP + p];
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m);
    if (lane == 0) partb[f] = s;
  }
}

struct Offs { int W[3], b[3]; };
struct CActs { const float* h[3]; };

template <int C, int F, int SD>
__global__ __launch_bounds__(kT) void k_encoder32_bwd(const float* __restrict__ x, const float* __restrict__ dfeat,
                                                      Ptrs w, CActs h, Offs off, long long total,
                                                      float* __restrict__ part) {
  using L0 = Lay<C, F, SD, 0>;
  using L1 = Lay<C, F, SD, 1>;
  using L2 = Lay<C, F, SD, 2>;
  constexpr int A = F * (L0::DP > L2::DP ? L0::DP : L2::DP), B = F * L1::DP;
  constexpr int IN = C * L0::PI > F * L1::PI ? C * L0::PI : F * L1::PI;
  __shared__ __attribute__((aligned(16))) float ra[A];      // D_2, then D_0
  __shared__ __attribute__((aligned(16))) float rb[B];      // D_1
  __shared__ __attribute__((aligned(16))) float rin[IN];    // the layer's input
  __shared__ float rw[F * L1::KR];
  __shared__ int2 tdx[9 * F];
  __shared__ int2 tdw[(L0::P + 3) / 4 * 4];
  constexpr int DX2 = (L2::PI + 15) / 16, DX1 = (L1::PI + 15) / 16;
  const int wave = threadIdx.x >> 6;
  const long long img = blockIdx.x;
  float* pp = part + img * total;

  Weights<L1, F> ww;
  ww.load(w.W[2]);
  zero4(ra, F * L2::DP);
  zero4(rb, F * L1::DP);
  copy4(h.h[1] + img * F * L1::P, rin, F * L1::P);
  ww.store(rw);
  ww.load(w.W[1]);
  fill_dx<L2, F>(tdx);
  fill_dw<L2>(tdw);
  __syncthreads();
  for (int e = threadIdx.x; e < F * L2::P; e += kT) {
    const int f = e / L2::P, p = e - f * L2::P, oy = p / L2::HO, ox = p - oy * L2::HO;
    const long long i = img * F * L2::P + e;
    ra[f * L2::DP + (oy + 2) * L2::DS + ox + 2] = h.h[2][i] > 0.f ? dfeat[i] : 0.f;
  }
  __syncthreads();
  db_sums<L2, F>(ra, pp + off.b[2]);
  for (int t = wave; t < DX2 + (L2::K + 15) / 16; t += kWaves) {
    if (t < DX2) dx_task<L2, L1, F>(t, ra, rw, tdx, rin, rb);
    else dw_task<L2, F>(t - DX2, ra, rin, tdw, pp + off.W[2]);
  }
  __syncthreads();
  copy4(h.h[0] + img * F * L0::P, rin, F * L0::P);
  ww.store(rw);
  fill_dx<L1, F>(tdx);
  fill_dw<L1>(tdw);
  __syncthreads();
  db_sums<L1, F>(rb, pp + off.b[1]);
  for (int t = wave; t < DX1 + (L1::K + 15) / 16; t += kWaves) {
    if (t < DX1) dx_task<L1, L0, F>(t, rb, rw, tdx, rin, ra);
    else dw_task<L1, F>(t - DX1, rb, rin, tdw, pp + off.W[1]);
  }
  __syncthreads();
  copy4(x + img * C * L0::PI, rin, C * L0::PI);
  fill_dw<L0>(tdw);
  __syncthreads();
  db_sums<L0, F>(ra, pp + off.b[0]);
  for (int t = wave; t < (L0::K + 15) / 16; t += kWaves) dw_task<L0, F>(t, ra, rin, tdw, pp + off.W[0]);
}

}  // namespace

bool encoder32_ok(int C, int F, int n_conv, int side) { return C == 9 && F == 32 && n_conv == 3 && side == 32; }

int encoder32_fwd(const float* x, int n, const float* const* W, const float* const* b, float* const* h,
                  float* xsave, float* feat2, hipStream_t st) {
  // copies take 16 bytes at a time; a caller's own image or feature buffer (the form
  // without a workspace) may be aligned to 4
  if (((uintptr_t)x | (uintptr_t)h[2]) % 16 != 0) return kNotApplicable;
  if (n <= 0) return SQ_OK;
  k_encoder32_fwd<9, 32, 32><<<n, kT, 0, st>>>(x, Ptrs{{W[0], W[1], W[2]}, {b[0], b[1], b[2]}},
                                               Acts{{h[0], h[1], h[2]}}, xsave, feat2);
  return launch_status("encoder32_fwd");
}

int encoder32_bwd(const float* x, int n, const float* dfeat, const float* const* W, const float* const* h,
                  const long long* Woff, const long long* boff, long long total, float* part, float* grad,
                  hipStream_t st) {
  if (n <= 0) return SQ_OK;
  Offs off;
  for (int i = 0; i < 3; ++i) {
    off.W[i] = (int)Woff[i];
    off.b[i] = (int)boff[i];
  }
  k_encoder32_bwd<9, 32, 32><<<n, kT, 0, st>>>(x, dfeat, Ptrs{{W[0], W[1], W[2]}, {nullptr, nullptr, nullptr}},
                                               CActs{{h[0], h[1], h[2]}}, off, total, part);
  SQ_TRY(launch_status("encoder32_bwd"));
  return encoder_reduce(part, n, total, grad, EncOrder{}, st);
}

}  // namespace sq
