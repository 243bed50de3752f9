// Dense eigenvector transforms on the matrix cores.
//
// With the full generalized eigenvectors of the periodised axis, K V = M V L
// and V^T M V = I (eqs. (EVP1a), (EVPcondA)), the 2D operator factors as
// A = (V^{-T} (x) I) (L (x) M_2 + I (x) (K_2 - w^2 M_2)) (V^{-1} (x) I), so
//   u = (V (x) I) blockdiag_l(T^A_l)^{-1} (V^T (x) I) f,
// the direct diagonalisation the paper writes in eq. (A2Dinv); in 3D the
// same holds with V_1 (x) V_2.  It needs no boundary steps at all; its cost
// is two dense transforms of 8 n flops per unknown each, which pays at small
// n where the transform is cheap and the three line passes of the fast
// method are not.
//
// The transform along the slow axis of a batch of [n][S] blocks,
//   out[b][m][x] (+)= sum_i Q[i][m] in[b][i][x],
// is a complex GEMM C = Q^T B on the matrix cores (cgemm.h).
#include "cgemm.h"

namespace helm {

namespace {

template <typename C> struct RealT;
template <> struct RealT<double2> { using T = double; };
template <> struct RealT<float2> { using T = float; };
template <typename R> struct CplxT;
template <> struct CplxT<double> { using T = double2; };
template <> struct CplxT<float> { using T = float2; };

template <typename R, typename TIN, typename TOUT, int T>
__global__ __launch_bounds__(256) void dense_kernel(DenseArgs a) {
  using G = CGemmTile<R, T>;
  __shared__ typename G::Lds lds;
  if (a.skip && *a.skip) return;
  const int n = a.n;
  const int64_t S = a.S;
  const int mt = (n + G::B - 1) / G::B;
  const int64_t xt = (S + G::B - 1) / G::B;
  int64_t blk = blockIdx.x;
  const int64_t xi = blk % xt;
  blk /= xt;
  const int mi = (int)(blk % mt);
  const int64_t beta = blk / mt;
  const int m0 = mi * G::B;
  const int64_t x0 = xi * G::B;
  const TIN* in = reinterpret_cast<const TIN*>(a.in) + beta * (int64_t)n * S;
  const typename CplxT<R>::T* Q = reinterpret_cast<const typename CplxT<R>::T*>(a.Q);  // [n][n]
  typename G::acc cr[T][T], ci[T][T];
  G::template run<false>(
      lds, n,
      // A[m][k] = Q[k][m], rows k of Q are contiguous in m
      [&](int k, int mm) { return Q[(int64_t)k * n + min(m0 + mm, n - 1)]; },
      // rows k of the input block, contiguous in x
      [&](int k, int xx) { return in[(int64_t)k * S + (x0 + xx < S ? x0 + xx : S - 1)]; },
      cr, ci);
  TOUT* out = reinterpret_cast<TOUT*>(a.out) + beta * (int64_t)n * S;
  G::each(cr, ci, [&](int mm, int xx, R re, R im) {
    const int m = m0 + mm;
    const int64_t x = x0 + xx;
    if (m < n && x < S) {
      double vr = (double)re * a.scale, vi = (double)im * a.scale;
      TOUT* o = out + (int64_t)m * S + x;
      if (a.accumulate) {
        vr += (double)o->x;
        vi += (double)o->y;
      }
      TOUT w;
      w.x = (typename RealT<TOUT>::T)vr;
      w.y = (typename RealT<TOUT>::T)vi;
      *o = w;
    }
  });
}

template <typename R, typename TIN, typename TOUT>
hipError_t launch_out(const DenseArgs& a, hipStream_t s) {
  auto blocks = [&](int64_t b) { return a.batch * ((a.n + b - 1) / b) * ((a.S + b - 1) / b); };
  const int64_t b64 = blocks(64), b32 = blocks(32);
  if (cgemm_tile(b64) == 1) {
    hipLaunchKernelGGL((dense_kernel<R, TIN, TOUT, 1>), dim3((unsigned)b32), dim3(256), 0, s, a);
  } else {
    if (b64 > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((dense_kernel<R, TIN, TOUT, 2>), dim3((unsigned)b64), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

template <typename R, typename TIN>
hipError_t launch_in(const DenseArgs& a, hipStream_t s) {
  return a.out_kind == ST_C64 ? launch_out<R, TIN, float2>(a, s) : launch_out<R, TIN, double2>(a, s);
}

}  // namespace

hipError_t launch_dense(const DenseArgs& a, bool fp32, hipStream_t s) {
  if (a.n < 1 || a.S < 1 || a.batch < 1 || !a.Q || !a.in || !a.out) return hipErrorInvalidValue;
  if (fp32) return a.in_kind == ST_C64 ? launch_in<float, float2>(a, s) : launch_in<float, double2>(a, s);
  return a.in_kind == ST_C64 ? launch_in<double, float2>(a, s) : launch_in<double, double2>(a, s);
}

}  // namespace helm
