// Complex matrix products on the matrix cores: the tile shared by the dense
// eigenvector transforms (dense.hip) and the modal transforms of the boundary
// steps (modal.hip).
//
// A 256-thread block computes a (32 T) x (32 T) tile of C = A B with real
// 16x16x4 MFMA operations, four real products per complex one; each of its
// four waves owns a quarter (T x T MFMA tiles, real and imaginary
// accumulators).  K steps of 16 are staged through two LDS buffers in planar
// (real / imaginary) form, padded against bank conflicts; one barrier per step
// separates the writes of a buffer from the reads of it two steps before.  The
// global loads of the next step (T = 2) or the next two (T = 1, whose products
// take less than a load) are in flight during a step's products: 257^2 dense
// mixed, products of 257 x 257 with 1028 columns, 18.3 -> 17.1 us and from
// complex128 input 27 -> 19 (its conversion had each load waited for); FP64 rows
// of 256^3 24 -> 21.5.
// T = 2 reuses every staged value twice as often; T = 1 gives four times the
// blocks for products that would leave compute units idle.
#pragma once

#include "helm_internal.h"

namespace helm {

constexpr int kGemmK = 16, kGemmPad = 4;

typedef double d4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

template <typename R> struct Mma;
// f64 16x16x4: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; output
// register r of lane l is D[l / 16 + 4 r][l % 16].
template <> struct Mma<double> {
  using acc = d4v;
  __device__ static acc op(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row(int lane, int r) { return lane / 16 + 4 * r; }
};
// f32 16x16x4: same operand layout; output register r of lane l is
// D[4 (l / 16) + r][l % 16].
template <> struct Mma<float> {
  using acc = f4v;
  __device__ static acc op(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row(int lane, int r) { return 4 * (lane / 16) + r; }
};

template <typename R, int T> struct CGemmTile {
  using M = Mma<R>;
  using acc = typename M::acc;
  static constexpr int B = 32 * T;                  // tile rows and columns
  static constexpr int kPer = kGemmK * B / 256;     // staged elements of each operand per thread
  struct Lds {
    R Ar[2][kGemmK][B + kGemmPad], Ai[2][kGemmK][B + kGemmPad], Br[2][kGemmK][B + kGemmPad], Bi[2][kGemmK][B + kGemmPad];
  };

  // la(k, m) and lb(k, x) load element (m, k) of A and (k, x) of B as a pair of
  // any real type, k < n, at tile-relative m and x; past the matrix they load any
  // element of it (that row or column of the tile is not used).  AROW:
  // consecutive threads load consecutive k of A (rows of A contiguous in k), else
  // consecutive m.  Loads are unconditional and converted where they are
  // staged: a load converted inside a branch is waited for there.
  template <bool AROW, class LA, class LB>
  __device__ static void run(Lds& s, int n, LA la, LB lb, acc (&cr)[T][T], acc (&ci)[T][T]) {
    constexpr int D = T == 1 ? 2 : 1;
    constexpr int KG = T == 1 ? 4 : 1;  // quarter steps whose operands are read ahead of the products
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int wm = (wv >> 1) * 16 * T, wn = (wv & 1) * 16 * T;
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int u = 0; u < T; ++u) {
        cr[t][u] = acc{0, 0, 0, 0};
        ci[t][u] = acc{0, 0, 0, 0};
      }
    decltype(la(0, 0)) qa[D][kPer];
    decltype(lb(0, 0)) qb[D][kPer];
    auto ka_of = [&](int t) { return AROW ? (tid + 256 * t) % kGemmK : (tid + 256 * t) / B; };
    auto ma_of = [&](int t) { return AROW ? (tid + 256 * t) / kGemmK : (tid + 256 * t) % B; };
    auto fetch = [&](int d, int k0) {
#pragma unroll
      for (int t = 0; t < kPer; ++t) {
        const int e = tid + 256 * t;
        qa[d][t] = la(min(k0 + ka_of(t), n - 1), ma_of(t));
        qb[d][t] = lb(min(k0 + e / B, n - 1), e % B);
      }
    };
    auto park = [&](int d, int k0, int buf) {
#pragma unroll
      for (int t = 0; t < kPer; ++t) {
        const int e = tid + 256 * t, ka = ka_of(t), ma = ma_of(t);
        const bool oka = k0 + ka < n, okb = k0 + e / B < n;
        s.Ar[buf][ka][ma] = oka ? (R)qa[d][t].x : R(0);
        s.Ai[buf][ka][ma] = oka ? (R)qa[d][t].y : R(0);
        s.Br[buf][e / B][e % B] = okb ? (R)qb[d][t].x : R(0);
        s.Bi[buf][e / B][e % B] = okb ? (R)qb[d][t].y : R(0);
      }
    };
    const int steps = (n + kGemmK - 1) / kGemmK;
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(d, d * kGemmK);
    park(0, 0, 0);
    if constexpr (T == 1) fetch(0, D * kGemmK);
    __syncthreads();
    auto step = [&](int d, int i) {
      const int buf = i & 1;
      if constexpr (T != 1) fetch(0, (i + 1) * kGemmK);
      R ar[KG][T], ai[KG][T], br[KG][T], bi[KG][T];
#pragma unroll
      for (int ks = 0; ks < kGemmK; ks += 4 * KG) {
#pragma unroll
        for (int q = 0; q < KG; ++q) {
          const int kl = ks + 4 * q + lane / 16, c16 = lane % 16;
#pragma unroll
          for (int t = 0; t < T; ++t) {
            ar[q][t] = s.Ar[buf][kl][wm + 16 * t + c16];
            ai[q][t] = s.Ai[buf][kl][wm + 16 * t + c16];
            br[q][t] = s.Br[buf][kl][wn + 16 * t + c16];
            bi[q][t] = s.Bi[buf][kl][wn + 16 * t + c16];
          }
        }
#pragma unroll
        for (int q = 0; q < KG; ++q)
#pragma unroll
          for (int t = 0; t < T; ++t)
#pragma unroll
            for (int u = 0; u < T; ++u) {
              cr[t][u] = M::op(ar[q][t], br[q][u], cr[t][u]);
              ci[t][u] = M::op(ar[q][t], bi[q][u], ci[t][u]);
              cr[t][u] = M::op(-ai[q][t], bi[q][u], cr[t][u]);
              ci[t][u] = M::op(ai[q][t], br[q][u], ci[t][u]);
            }
      }
      // (unconditional, so that the number of loads in flight is known where
      // one is waited for; past the end zeros go to a buffer not read again)
      park((d + 1) % D, (i + 1) * kGemmK, buf ^ 1);
      if constexpr (T == 1) fetch((d + 1) % D, (i + 1 + D) * kGemmK);
      __syncthreads();
    };
    // (no exit from inside the loop: it would make every wait in it one for all
    // loads)
    int i = 0;
    for (; i + D <= steps; i += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) step(d, i + d);
    }
#pragma unroll
    for (int d = 0; d + 1 < D; ++d)
      if (i + d < steps) step(d, i + d);
  }

  // st(m, x, re, im) for every element of the block's tile this thread holds.
  template <class ST> __device__ static void each(const acc (&cr)[T][T], const acc (&ci)[T][T], ST st) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int wm = (wv >> 1) * 16 * T, wn = (wv & 1) * 16 * T;
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int u = 0; u < T; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          st(wm + 16 * t + M::row(lane, r), wn + 16 * u + lane % 16, cr[t][u][r], ci[t][u][r]);
  }
};

// Tile of a product with `b64` blocks of 64 x 64: the small one while the large
// one leaves compute units without a block.
inline int cgemm_tile(int64_t b64) { return b64 < 256 ? 1 : 2; }

}  // namespace helm
