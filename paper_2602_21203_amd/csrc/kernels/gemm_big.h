// The 64 x 64 tile of the plain-matrix products (included by gemm.hip, after the
// operand and store types it shares with the 32 x 32 tile).
//
// The 32 x 32 tile gives small products enough workgroups and a short K chain per
// wave, but it reads each operand M / 32 or N / 32 times, and a large product is
// bound by those L2 reads.  Here a 256-thread workgroup owns a 64 x 64 tile: the
// operands' 32 k of a stage are loaded once, coalesced, into registers stages
// ahead, and stored to one of two LDS buffers as [row][k] (rows padded so that
// 16-byte reads and writes of neighbouring rows fall on different banks); each wave
// contracts all of K for its 32 x 32 quadrant.  Half the operand bytes, one barrier
// per 32 k.
//
// The arithmetic is the 32 x 32 tile's bit for bit: there four waves contract a
// quarter of K each and their sums are added in order, so here the accumulator is
// added to a running sum, and cleared, at the same quarter boundaries; chunks of
// 32 k, the k of each lane in a chunk and the MFMA order are the same too.
//
// The loop is written for few instructions and registers (four workgroups share a
// compute unit): every address is a uniform base (scalar registers) plus a 32-bit
// offset per thread, and loads past the end are clamped rather than skipped, so
// that waiting for one stage leaves the later ones in flight.
#pragma once

namespace sq {

constexpr int kBigTile = 64;
constexpr int kBigK = 32;   // k per stage: one chunk (kRKC)

template <bool BF16> struct BigLds {
  using T = typename RLds<BF16>::T;
  static constexpr int LD = BF16 ? kBigK + 8 : kBigK + 4;   // row stride (elements)
  static constexpr int OP = kBigTile * LD;                  // one operand's stage
  static constexpr int BYTES = 2 * 2 * OP * (int)sizeof(T);
};

// How an FP32 operand's stage is read.  kBigCol: lanes along rows, any strides (the
// rows contiguous in the products that use it), 8 consecutive k per thread.
// kBigRow: k-contiguous rows, 16-byte aligned.  kBigRow1: k-contiguous rows at any
// alignment (weights in the flat parameter vector), lanes along k.
// kBigCol4: rows contiguous and 16-byte aligned at every k: four rows at four
// consecutive k per thread (a 4 x 4 block, transposed in registers).
enum { kBigCol = 0, kBigRow = 1, kBigRow1 = 2, kBigCol4 = 3 };

// element of type T at a uniform base plus a per-thread byte offset
template <class T>
__device__ __forceinline__ T big_ld(const void* base, unsigned off) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + off);
}

template <bool BF16>
__device__ __forceinline__ void big_put8(const float* v, typename BigLds<BF16>::T* dst) {
  if constexpr (BF16) {
    bf16x8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (__bf16)v[e];
    *reinterpret_cast<bf16x8*>(dst) = h;
  } else {
    *reinterpret_cast<f4v*>(dst) = f4v{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f4v*>(dst + 4) = f4v{v[4], v[5], v[6], v[7]};
  }
}

// the base and the k range of a stage: a k-concatenated operand's second part starts
// at kalt (a multiple of the stage)
template <class P> struct BigAt { P base; int k0, kend; };
template <class P>
__device__ __forceinline__ BigAt<P> big_at(P base, P kbase, int stage, int K, int kalt) {
  const int k0 = stage * kBigK;
  return k0 >= kalt ? BigAt<P>{kbase, k0 - kalt, K - kalt} : BigAt<P>{base, k0, K};
}

// A stage (64 rows x 32 k) of an FP32 operand.  load() only requests it: rows and k
// past the end are clamped into the matrix, so nothing waits for a value; store()
// then writes zeros for the k past the end (rows past the end give results that are
// not stored).
template <bool BF16, int KIND> struct BigF {
  using LL = BigLds<BF16>;
  using T = typename LL::T;
  using Regs = float[8];
  const float* base; const float* kbase; long long lr, lk; int kalt, r0, rows, K;
  unsigned off[2];   // this thread's byte offsets
  int wave;
  __device__ __forceinline__ BigF(const RMat& a, int z, int r0_, int rows_, int K_)
      : base(a.batch(z)), kbase(a.kp ? a.kp + (long long)z * a.sz : nullptr), lr(a.lr), lk(a.lk), kalt(a.kalt),
        r0(r0_), rows(rows_), K(K_), wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
    const int t = threadIdx.x;
    if constexpr (KIND == kBigCol) {
      off[0] = (unsigned)min(r0 + (t & 63), rows - 1) * (unsigned)(4 * lr);
    } else if constexpr (KIND == kBigRow) {
#pragma unroll
      for (int j = 0; j < 2; ++j) off[j] = (unsigned)min(r0 + 32 * j + (t >> 3), rows - 1) * (unsigned)(4 * lr);
    } else if constexpr (KIND == kBigCol4) {
      off[0] = 4u * (unsigned)min(r0 + 4 * (t & 15), (rows - 1) & ~3);   // (a group holding a valid row)
    }
  }
  // k of element i of this thread's registers, within the stage
  __device__ __forceinline__ int kof(int i) const {
    const int t = threadIdx.x;
    if constexpr (KIND == kBigCol) return 8 * wave + i;
    if constexpr (KIND == kBigRow) return 4 * (t & 7) + (i & 3);
    if constexpr (KIND == kBigCol4) return 2 * (t >> 4) + (i >> 2);
    return t & 31;
  }
  __device__ __forceinline__ void load(int stage, Regs& v) const {
    const auto g = big_at(base, kbase, stage, K, kalt);
    const int t = threadIdx.x, last = g.kend - 1 - g.k0;   // last k of the stage, counted from its first
    if constexpr (KIND == kBigCol) {
      const float* q = g.base + (long long)g.k0 * lk;
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = big_ld<float>(q + min(8 * wave + i, last) * lk, off[0]);
    } else if constexpr (KIND == kBigCol4) {
      const float* q = g.base + (long long)g.k0 * lk;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f4v x = big_ld<f4v>(q, off[0] + (unsigned)min(2 * (t >> 4) + j, last) * (unsigned)(4 * lk));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * j + e] = x[e];
      }
    } else if constexpr (KIND == kBigRow) {
      // the 16-byte group of the last k may hold elements past the end: same aligned
      // group, so mapped memory, and store() drops them
      const unsigned kq = 4u * (unsigned)min(4 * (t & 7), last & ~3);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f4v x = big_ld<f4v>(g.base + g.k0, off[j] + kq);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * j + e] = x[e];
      }
    } else {
      const unsigned kq = 4u * (unsigned)min(t & 31, last);
      const float* q = g.base + g.k0;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        v[j] = big_ld<float>(q, (unsigned)min(r0 + 8 * j + (t >> 5), rows - 1) * (unsigned)(4 * lr) + kq);
    }
  }
  template <bool MASK> __device__ __forceinline__ void store(int stage, const Regs& r, T* lds) const {
    const int t = threadIdx.x;
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = r[i];
    if constexpr (MASK) {
      const auto g = big_at(base, kbase, stage, K, kalt);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = g.k0 + kof(i) < g.kend ? v[i] : 0.f;
    }
    if constexpr (KIND == kBigCol) {
      big_put8<BF16>(v, lds + (t & 63) * LL::LD + 8 * (t >> 6));
    } else if constexpr (KIND == kBigRow) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        T* dst = lds + (32 * j + (t >> 3)) * LL::LD + 4 * (t & 7);
        if constexpr (BF16) {
          bf16x4 h;
#pragma unroll
          for (int e = 0; e < 4; ++e) h[e] = (__bf16)v[4 * j + e];
          *reinterpret_cast<bf16x4*>(dst) = h;
        } else {
          *reinterpret_cast<f4v*>(dst) = f4v{v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]};
        }
      }
    } else if constexpr (KIND == kBigCol4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        T* dst = lds + (4 * (t & 15) + e) * LL::LD + 2 * (t >> 4);
        typedef T t2 __attribute__((ext_vector_type(2)));
        *reinterpret_cast<t2*>(dst) = t2{(T)v[e], (T)v[4 + e]};
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) lds[(8 * j + (t >> 5)) * LL::LD + (t & 31)] = (T)v[j];
    }
  }
  // the fragments of rows row0 .. row0 + 31
  static __device__ __forceinline__ void frag(const T* lds, int row0, int li, int lq, RFrag<BF16>& f) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const T* src = lds + (row0 + 16 * i + li) * LL::LD + 8 * lq;
      if constexpr (BF16) {
        f.v[i] = *reinterpret_cast<const bf16x8*>(src);
      } else {
        const f4v a = *reinterpret_cast<const f4v*>(src), b = *reinterpret_cast<const f4v*>(src + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          f.v[i][e] = a[e];
          f.v[i][4 + e] = b[e];
        }
      }
    }
  }
};

// a stage of an operand's bfloat16 copy, 16 bytes per thread: plain rows in groups of
// 8 k, kept as [row][k]; transposed (TR) 8 rows at one k, kept as [k][row] and read
// back transposed
template <bool TR> struct BigH {
  using T = __bf16;
  using Regs = u4v;
  static constexpr int LD = TR ? kBigTile + 8 : BigLds<true>::LD;
  static_assert(!TR || kBigK * LD <= BigLds<true>::OP, "the transposed stage fits its operand's buffer");
  const uint16_t* base; const uint16_t* kbase; long long ld; int kalt, lim, K;
  unsigned off;
  __device__ __forceinline__ BigH(const HMat& a, int z, int r0, int rows, int K_)
      : base(a.batch(z)), kbase(a.kp ? a.kp + (long long)z * a.sz : nullptr), ld(a.ld), kalt(a.kalt), lim(a.lim),
        K(K_) {
    const int t = threadIdx.x;
    if constexpr (TR) off = 2u * (unsigned)min(r0 + 8 * (t & 7), lim);   // a group inside the line
    else off = (unsigned)min(r0 + (t >> 2), rows - 1) * (unsigned)(2 * ld);
  }
  __device__ __forceinline__ void load(int stage, Regs& v) const {
    const auto g = big_at(base, kbase, stage, K, kalt);
    const int t = threadIdx.x;
    if constexpr (TR)
      v = big_ld<u4v>(g.base + (long long)g.k0 * ld,
                      off + (unsigned)min(t >> 3, g.kend - 1 - g.k0) * (unsigned)(2 * ld));
    else
      v = big_ld<u4v>(g.base + g.k0, off + 2u * (unsigned)min(8 * (t & 3), lim - g.k0));
  }
  template <bool MASK> __device__ __forceinline__ void store(int stage, const Regs& r, T* lds) const {
    const int t = threadIdx.x;
    u4v v = r;
    if constexpr (MASK) {
      const auto g = big_at(base, kbase, stage, K, kalt);
      if constexpr (TR) v = g.k0 + (t >> 3) < g.kend ? v : u4v{0u, 0u, 0u, 0u};
      else v = hmask(v, g.k0 + 8 * (t & 3), g.kend);
    }
    if constexpr (TR) *reinterpret_cast<u4v*>(lds + (t >> 3) * LD + 8 * (t & 7)) = v;
    else *reinterpret_cast<u4v*>(lds + (t >> 2) * LD + 8 * (t & 3)) = v;
  }
  // the fragments of rows row0 .. row0 + 31
  static __device__ __forceinline__ void frag(const T* lds, int row0, int li, int lq, RFrag<true>& f) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if constexpr (TR) {
        const T* p = lds + (8 * lq + (li >> 2)) * LD + row0 + 16 * i + 4 * (li & 3);
        f.v[i] = lds_tr8(p, p + 4 * LD);
      } else {
        f.v[i] = *reinterpret_cast<const bf16x8*>(lds + (row0 + 16 * i + li) * LD + 8 * lq);
      }
    }
  }
};

// a wave's 32 x 32 quadrant at (r0, c0): StMat::put for each element, its uniform
// choices outside the element loop
__device__ __forceinline__ void big_put(const StMat& st, v4f (&v)[2][2], int M, int N, int r0, int c0, int z, int li,
                                        int lq) {
  const float* bias = st.bias ? (z < st.bias_zalt ? st.bias + z * st.bias_sz
                                                  : st.bias_alt + (z - st.bias_zalt) * st.bias_sz)
                              : nullptr;
  float* base = st.p + z * st.sz;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int c = c0 + 16 * j + li;
    if (c >= N) continue;
    if (bias) {
      const float bv = bias[c];
#pragma unroll
      for (int i = 0; i < 2; ++i) v[i][j] += bv;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = r0 + 16 * i + 4 * lq + q;
        float* p = base + (long long)r * st.ld + c;
        float x = v[i][j][q];
        if (r >= M) continue;
        if (st.acc) x += *p;
        if (st.relu) x = fmaxf(x, 0.f);
        *p = x;
      }
  }
}

// LDS hand-over between the waves: their LDS operations complete, their global
// loads stay in flight (the builtins, so that the compiler knows what has been waited for)
__device__ __forceinline__ void big_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// one 64 x 64 output tile (bx, by) of batch z; K > 0.  Two stages of both operands
// are in flight (register slot = LDS buffer = stage parity).
template <bool BF16, class OA, class OB>
__device__ __forceinline__ void big_tile(const OA& a, const OB& b, const StMat& st, int M, int N, int K, int bx,
                                         int by, int z, char* ldsb) {
  static_assert(kBigK == kRKC, "one chunk per stage");
  using LL = BigLds<BF16>;
  using T = typename LL::T;
  T* lds = reinterpret_cast<T*>(ldsb);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lq = lane >> 4;
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
  const int per = ((K + 3) / 4 + kRKC - 1) / kRKC;            // chunks of a quarter
  const int ns = (K + kBigK - 1) / kBigK;                     // stages

  v4f acc[2][2], tot[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = tot[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  int in_q = 0, quarters = 0;   // chunks of the current quarter, quarters finished
  auto fold = [&] {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        tot[i][j] = quarters == 0 ? acc[i][j] : tot[i][j] + acc[i][j];
        acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
      }
    in_q = 0;
    ++quarters;
  };

  typename OA::Regs ra[2];
  typename OB::Regs rb[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    a.load(min(u, ns - 1), ra[u]);
    b.load(min(u, ns - 1), rb[u]);
    __builtin_amdgcn_sched_barrier(0);   // requested in stage order
  }
  RFrag<BF16> fa[2], fb[2];   // a stage's fragments, read one stage ahead
  // stage s (slot u): read the next stage's fragments, store the stage after that,
  // request another, and multiply
  auto turn = [&](int s, auto uc, auto mask) {
    constexpr int u = decltype(uc)::value;
    constexpr bool MASK = decltype(mask)::value;
    T* cur = lds + (u & 1) * 2 * LL::OP;
    const T* nxt = lds + ((u + 1) & 1) * 2 * LL::OP;
    big_barrier();   // stage s + 1 is in LDS, and everybody has read stage s
    OA::frag(nxt, wm, li, lq, fa[(u + 1) & 1]);
    OB::frag(nxt + LL::OP, wn, li, lq, fb[(u + 1) & 1]);
    a.template store<MASK>(min(s + 2, ns - 1), ra[u], cur);
    b.template store<MASK>(min(s + 2, ns - 1), rb[u], cur + LL::OP);
    a.load(min(s + 4, ns - 1), ra[u]);
    b.load(min(s + 4, ns - 1), rb[u]);
    rmma<BF16>(fa[u & 1], fb[u & 1], acc);
    if (++in_q == per) fold();
  };
  using U0 = std::integral_constant<int, 0>;
  using U1 = std::integral_constant<int, 1>;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    T* cur = lds + u * 2 * LL::OP;
    a.template store<true>(min(u, ns - 1), ra[u], cur);
    b.template store<true>(min(u, ns - 1), rb[u], cur + LL::OP);
    a.load(min(u + 2, ns - 1), ra[u]);
    b.load(min(u + 2, ns - 1), rb[u]);
    __builtin_amdgcn_sched_barrier(0);
    if (u == 0) {
      big_barrier();
      OA::frag(lds, wm, li, lq, fa[0]);
      OB::frag(lds + LL::OP, wn, li, lq, fb[0]);
    }
  }
  int s = 0;
  for (; (s + 4) * kBigK <= K; s += 2) {   // the stages stored here (s + 2, s + 3) are whole
    turn(s, U0{}, std::false_type{});
    turn(s + 1, U1{}, std::false_type{});
  }
  for (; s < ns; s += 2) {
    turn(s, U0{}, std::true_type{});
    if (s + 1 < ns) turn(s + 1, U1{}, std::true_type{});
  }
  while (quarters < 4) fold();   // the last quarter, and empty ones (adding zero, as their waves would)
  big_put(st, tot, M, N, bx * kBigTile + wm, by * kBigTile + wn, z, li, lq);
}

template <bool BF16, int KA, int KB>
__device__ __forceinline__ void big_tile_f(const RMat& a, const RMat& b, const StMat& st, int M, int N, int K, int bx,
                                           int by, int z, char* lds) {
  big_tile<BF16>(BigF<BF16, KA>(a, z, bx * kBigTile, M, K), BigF<BF16, KB>(b, z, by * kBigTile, N, K), st, M,
                          N, K, bx, by, z, lds);
}
template <bool TA, bool TB>
__device__ __forceinline__ void big_tile_h(const HMat& a, const HMat& b, const StMat& st, int M, int N, int K, int bx,
                                           int by, int z, char* lds) {
  big_tile<true>(BigH<TA>(a, z, bx * kBigTile, M, K), BigH<TB>(b, z, by * kBigTile, N, K), st, M, N, K, bx,
                          by, z, lds);
}

template <bool BF16, int KA, int KB>
__global__ __launch_bounds__(kThreads, BF16 ? 4 : 3) void k_gemm_big(RMat a, RMat b, StMat st, int M, int N, int K) {
  __shared__ __attribute__((aligned(16))) char lds[BigLds<BF16>::BYTES];
  int bx, by, bz;
  tile_of(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), gridDim.x, gridDim.y, gridDim.z, bx, by,
          bz);
  big_tile_f<BF16, KA, KB>(a, b, st, M, N, K, bx, by, bz, lds);
}

template <bool TA, bool TB>
__global__ __launch_bounds__(kThreads, 4) void k_gemm_big_h(HMat a, HMat b, StMat st, int M, int N, int K) {
  __shared__ __attribute__((aligned(16))) char lds[BigLds<true>::BYTES];
  int bx, by, bz;
  tile_of(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z), gridDim.x, gridDim.y, gridDim.z, bx, by,
          bz);
  big_tile_h<TA, TB>(a, b, st, M, N, K, bx, by, bz, lds);
}

}  // namespace sq
