// Complex matrix products on the matrix cores: the tile shared by the dense
// eigenvector transforms (dense.hip) and the modal transforms of the boundary
// steps (modal.hip).
//
// A 256-thread block computes a (32 T) x (32 T) tile of C = A B with real
// 16x16x4 MFMA operations, four real products per complex one; each of its
// four waves owns a quarter (T x T MFMA tiles, real and imaginary
// accumulators).  K steps of 16 are staged through two LDS buffers in planar
// (real / imaginary) form, padded against bank conflicts, with the next step's
// global loads in flight during the current step's products; one barrier per
// step separates the writes of a buffer from the reads of it two steps before.
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

  // la(k, m, re, im) and lb(k, x, re, im) load element (m, k) of A and (k, x)
  // of B, tile-relative m and x, zero outside; k < n.  AROW: consecutive
  // threads load consecutive k of A (rows of A contiguous in k), else
  // consecutive m.
  template <bool AROW, class LA, class LB>
  __device__ static void run(Lds& s, int n, LA la, LB lb, acc (&cr)[T][T], acc (&ci)[T][T]) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int wm = (wv >> 1) * 16 * T, wn = (wv & 1) * 16 * T;
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int u = 0; u < T; ++u) {
        cr[t][u] = acc{0, 0, 0, 0};
        ci[t][u] = acc{0, 0, 0, 0};
      }
    R qa[kPer][2], qb[kPer][2];
    auto fetch = [&](int k0) {
#pragma unroll
      for (int t = 0; t < kPer; ++t) {
        const int e = tid + 256 * t;
        const int ka = AROW ? e % kGemmK : e / B, ma = AROW ? e / kGemmK : e % B;
        qa[t][0] = qa[t][1] = 0;
        if (k0 + ka < n) la(k0 + ka, ma, qa[t][0], qa[t][1]);
        const int kb = e / B, xb = e % B;
        qb[t][0] = qb[t][1] = 0;
        if (k0 + kb < n) lb(k0 + kb, xb, qb[t][0], qb[t][1]);
      }
    };
    auto park = [&](int buf) {
#pragma unroll
      for (int t = 0; t < kPer; ++t) {
        const int e = tid + 256 * t;
        const int ka = AROW ? e % kGemmK : e / B, ma = AROW ? e / kGemmK : e % B;
        s.Ar[buf][ka][ma] = qa[t][0];
        s.Ai[buf][ka][ma] = qa[t][1];
        s.Br[buf][e / B][e % B] = qb[t][0];
        s.Bi[buf][e / B][e % B] = qb[t][1];
      }
    };
    fetch(0);
    park(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < n; k0 += kGemmK) {
      const bool more = k0 + kGemmK < n;
      if (more) fetch(k0 + kGemmK);
#pragma unroll
      for (int ks = 0; ks < kGemmK; ks += 4) {
        const int kl = ks + lane / 16, c16 = lane % 16;
        R ar[T], ai[T], an[T], br[T], bi[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
          ar[t] = s.Ar[buf][kl][wm + 16 * t + c16];
          ai[t] = s.Ai[buf][kl][wm + 16 * t + c16];
          an[t] = -ai[t];
          br[t] = s.Br[buf][kl][wn + 16 * t + c16];
          bi[t] = s.Bi[buf][kl][wn + 16 * t + c16];
        }
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
          for (int u = 0; u < T; ++u) {
            cr[t][u] = M::op(ar[t], br[u], cr[t][u]);
            cr[t][u] = M::op(an[t], bi[u], cr[t][u]);
            ci[t][u] = M::op(ar[t], bi[u], ci[t][u]);
            ci[t][u] = M::op(ai[t], br[u], ci[t][u]);
          }
      }
      if (more) park(buf ^ 1);
      __syncthreads();
      buf ^= 1;
    }
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
