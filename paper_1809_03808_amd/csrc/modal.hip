// Boundary steps of a 3D solve in the eigenbasis of the last axis.
//
// With the generalized eigenvectors of the last axis, K_3 V = M_3 V L and
// V^T M_3 V = I (eqs. (EVP1a), (EVPcondA) for that axis), every line matrix of
// the method is diagonal, V^T (s M_3 + K_3) V = s + L, whatever its mode.  A
// boundary vector held as v = V a (a = V^T M_3 v) therefore goes through the
// boundary steps one component p at a time:
//   C_2(l) v                 ->  A_2(l, p) a,  A_2 = dK_2 + (s_l + lambda_p) dM_2  (2 x 2)
//   inner Step 2 of mode l   ->  S(l, p) = sum_m v_m v_m^T / (s_lm + lambda_p)      (2 x 2)
//   outer Step 2 of mode m   ->  H(m, p) = sum_l v_l v_l^T / (s_lm + lambda_p)      (2 x 2)
//   sweeps of right-hand sides generated from boundary vectors (Steps 2 and 3,
//   eqs. (step2-1), (step3term)), reduced again (eqs. (2dBs1), (step2-3))
//                            ->  sums over l or m of weights / (s_lm + lambda_p).
// Of the nine line sweeps of a 3D solve this leaves the three that involve the
// N-sized right-hand side itself: its two reductions (over the inner and over
// the outer modes) and the storing sweep of Step 3.  S and H are precomputed
// per plan (3 (n1 + n2) n3 values); the sums over modes are evaluated in every
// solve, each denominator formed in registers, about 26 FP64 instructions per
// denominator and right-hand side against about 90 per unknown of a sweep, and
// a quarter of the denominators, because s_lm is even in both modes.
#include "cgemm.h"

namespace helm {

namespace {

// ---------------------------------------------------------------------------
// Partial sums of the two reducing sweeps: out[g][r] = sum_t in[g][t][r] over
// 2 nL values r.  A block takes 64 consecutive r of a group; its waves take
// interleaved tiles t, so that the few groups of a small grid with many tiles
// (129^3: 34 groups of 31 tiles) still keep enough loads in flight (summed by
// the product's own loads of its A operand: 142 us there, 5 + 14 us this way).
// ---------------------------------------------------------------------------
constexpr int kGatherWaves = 4;

__global__ __launch_bounds__(64 * kGatherWaves) void modal_gather_kernel(const double2* __restrict__ p0, int64_t g0,
                                                                         int nt0, double2* __restrict__ o0,
                                                                         const double2* __restrict__ p1, int nt1,
                                                                         double2* __restrict__ o1, int nL,
                                                                         const int* skip) {
  __shared__ double2 sm[kGatherWaves][64];
  if (skip && *skip) return;
  const int per = 2 * nL, ct = (per + 63) / 64;
  int64_t g = blockIdx.x / ct;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r = (int)(blockIdx.x % ct) * 64 + lane;
  const bool second = g >= g0;
  if (second) g -= g0;
  const double2* p = second ? p1 : p0;
  double2* o = second ? o1 : o0;
  const int nt = second ? nt1 : nt0;
  double2 s = make_double2(0, 0);
  if (r < per)
    for (int t = wv; t < nt; t += kGatherWaves) s = cadd(s, p[(g * nt + t) * per + r]);
  sm[wv][lane] = s;
  __syncthreads();
  if (wv == 0 && r < per) {
    for (int w = 1; w < kGatherWaves; ++w) s = cadd(s, sm[w][lane]);
    o[g * per + r] = s;
  }
}

// ---------------------------------------------------------------------------
// Rows of boundary vectors times an nL x nL matrix: the modal transform of the
// reduced boundary values and its transpose, the generated rows of Step 3.
// Bound by the FP64 matrix rate at many right-hand sides (512^3 x 4: 17.2
// GFLOP in 350 us, 49 TFLOP/s), by latency at few.
// ---------------------------------------------------------------------------
template <int T>
__global__ __launch_bounds__(256) void modal_rows_kernel(const double2* __restrict__ Q, int nL, int nb, ModalRows s0,
                                                         ModalRows s1, int tiles0, const int* skip) {
  using G = CGemmTile<double, T>;
  __shared__ typename G::Lds lds;
  if (skip && *skip) return;
  const int xt = (nL + G::B - 1) / G::B;
  int rt = (int)(blockIdx.x / xt);
  const int x0 = (int)(blockIdx.x % xt) * G::B;
  const bool second = rt >= tiles0;
  const ModalRows s = second ? s1 : s0;
  if (second) rt -= tiles0;
  const int64_t rows = 2 * (int64_t)nb * s.n, r0 = (int64_t)rt * G::B;
  typename G::acc cr[T][T], ci[T][T];
  G::template run<true>(
      lds, nL,
      [&](int k, int mm) { return s.in[(r0 + mm < rows ? r0 + mm : rows - 1) * nL + k]; },
      [&](int k, int xx) { return Q[(int64_t)k * nL + min(x0 + xx, nL - 1)]; },
      cr, ci);
  G::each(cr, ci, [&](int mm, int xx, double re, double im) {
    const int64_t r = r0 + mm;
    const int x = x0 + xx;
    if (r < rows && x < nL) {
      const int64_t bg = r >> 1, b = bg / s.n, g = bg - b * s.n;
      const int64_t o = b * s.ob + g * s.og + (r & 1) * s.ok + x;
      if (s.out_c64) reinterpret_cast<float2*>(s.out)[o] = make_float2((float)re, (float)im);
      else reinterpret_cast<double2*>(s.out)[o] = make_double2(re, im);
    }
  });
}

// q = A (a + S A a) for one (mode, p): the boundary operator, Step 2 and the
// boundary operator again, with A = dK + (s + lambda_p) dM.
struct MidOp {
  double2 A[2][2], S00, S01, S11;
};
__device__ inline MidOp mid_op(const ModalMid& m, int g, int nL, int p, double2 lam) {
  MidOp o;
  const double2 s = cadd(m.sO[g], lam);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      o.A[i][j] = make_double2(fma(s.x, m.d.dM[i][j], m.d.dK[i][j].x), fma(s.y, m.d.dM[i][j], m.d.dK[i][j].y));
  const double2* t = m.tab + (int64_t)g * 3 * nL + p;
  o.S00 = t[0];
  o.S01 = t[nL];
  o.S11 = t[2 * nL];
  return o;
}
__device__ inline void mid_apply(const MidOp& o, double2& a0, double2& a1) {
  const double2 r0 = cfma(o.A[0][0], a0, cmul(o.A[0][1], a1)), r1 = cfma(o.A[1][0], a0, cmul(o.A[1][1], a1));
  const double2 w0 = cfma(o.S00, r0, cfma(o.S01, r1, a0)), w1 = cfma(o.S01, r0, cfma(o.S11, r1, a1));
  a0 = cfma(o.A[0][0], w0, cmul(o.A[0][1], w1));
  a1 = cfma(o.A[1][0], w0, cmul(o.A[1][1], w1));
}

__global__ __launch_bounds__(256) void modal_mid_kernel(ModalMid m, int nb, int nG, int nL, const double2* lam,
                                                        const double2* __restrict__ in, double2* out,
                                                        const int* skip) {
  if (skip && *skip) return;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)nb * nG * nL) return;
  const int64_t bg = i / nL;
  const int p = (int)(i - bg * nL), g = (int)(bg % nG);
  double2 a0 = in[bg * 2 * nL + p], a1 = in[bg * 2 * nL + nL + p];
  mid_apply(mid_op(m, g, nL, p, lam[p]), a0, a1);
  out[bg * 2 * nL + p] = a0;
  out[bg * 2 * nL + nL + p] = a1;
}

// ---------------------------------------------------------------------------
// Sums over the modes s of one direction for every mode g of the other:
//   Y[r][j] = sum_s rho_r[s] X_j[s] / (sigma_gs + lambda_p),
//   out_r[g] = add_r[g] + gen_0[g] Y[r][0] + gen_1[g] Y[r][1],
// rho_0 = 1/nS, rho_1 = e^{-i theta_s}/nS, sigma real and even in s and in g
// (the periodic branches of both directions).  The denominators of s and
// nS - s are equal, so their two terms are added before the division, and the
// Y of g serve nG - g as well.  Lanes run over p; the waves of a block take
// interleaved s for the same (p, g) tile, so that even one right-hand side of a
// small grid has enough waves, and add their sums through LDS.  A block holds
// TG modes g of NB right-hand sides: X is read once per TG modes, a
// denominator serves NB right-hand sides (TG x NB = 4 keeps the 16
// accumulators in registers).  Bound by FP64 issue.
// ---------------------------------------------------------------------------
constexpr int kSumWaves = 8;

template <int TG, int NB>
__global__ __launch_bounds__(64 * kSumWaves) void modal_sum_kernel(ModalSum a) {
  constexpr int NV = TG * NB * 4;
  __shared__ double2 part[kSumWaves / 2][NV][64];
  if (a.skip && *a.skip) return;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nL = a.nL, nS = a.nS, nG = a.nG;
  const int pt = (nL + 63) / 64, gt = (nG / 2 + TG) / TG;  // g = 0 ... nG / 2
  int64_t blk = blockIdx.x;
  const int p = (int)(blk % pt) * 64 + lane;
  blk /= pt;
  const int g0 = (int)(blk % gt) * TG;
  const int b0 = (int)(blk / gt) * NB;
  const bool ok = p < nL;
  const int pc = ok ? p : nL - 1;
  const double2 lam = a.lam[pc], lamlo = a.lamlo[pc];
  const double li = lam.y + lamlo.y, li2 = li * li;
  double2 acc[NB][TG][2][2];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int t = 0; t < TG; ++t)
#pragma unroll
      for (int r = 0; r < 2; ++r) acc[b][t][r][0] = acc[b][t][r][1] = make_double2(0, 0);
  for (int s = wv; 2 * s <= nS; s += kSumWaves) {
    const int sp = s == 0 ? 0 : nS - s;
    const bool pair = sp != s;
    const double2 w = a.rho1[s];
    double2 x[NB][2][2];  // [b][r][j]: the two terms of the pair, weighted by rho_r (rho_0 without 1/nS)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int bb = b0 + b < a.nb ? b0 + b : a.nb - 1;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const double2 u = a.X[(((int64_t)bb * nS + s) * 2 + j) * nL + pc];
        double2 v = a.X[(((int64_t)bb * nS + sp) * 2 + j) * nL + pc];
        if (!pair) v = make_double2(0, 0);
        x[b][0][j] = cadd(u, v);
        x[b][1][j] = cfma(w, u, cmul(make_double2(w.x, -w.y), v));
      }
    }
#pragma unroll
    for (int t = 0; t < TG; ++t) {
      const int g = min(g0 + t, nG / 2);
      const double dr = (a.sig[s * a.sS + g * a.sG].x + lam.x) + lamlo.x;
      const double ri = rcp_nr(fma(dr, dr, li2));
      const double2 D = make_double2(dr * ri, -li * ri);
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[b][t][r][j] = cfma(D, x[b][r][j], acc[b][t][r][j]);
    }
  }
  // sum over the waves: the upper half of them hands its sums to the lower half
#pragma unroll
  for (int h = kSumWaves / 2; h > 0; h >>= 1) {
    if (wv >= h && wv < 2 * h) {
#pragma unroll
      for (int i = 0; i < NV; ++i) part[wv - h][i][lane] = (&acc[0][0][0][0])[i];
    }
    __syncthreads();
    if (wv < h) {
#pragma unroll
      for (int i = 0; i < NV; ++i) (&acc[0][0][0][0])[i] = cadd((&acc[0][0][0][0])[i], part[wv][i][lane]);
    }
    __syncthreads();
  }
  if (wv != 0 || !ok) return;
  const double inv = 1.0 / nS;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    if (b0 + b >= a.nb) break;
#pragma unroll
    for (int t = 0; t < TG; ++t) {
      const int g = g0 + t;
      if (2 * g > nG) break;
      for (int half = 0; half < 2; ++half) {
        const int gg = half ? nG - g : g;
        if (half && (g == 0 || gg == g)) break;
        const double2 e0 = a.gen0[gg], e1 = a.gen1[gg];
        const int64_t o = ((int64_t)(b0 + b) * nG + gg) * 2 * nL + p;
        double2 v0 = cfma(e0, cscale(acc[b][t][0][0], inv), cfma(e1, cscale(acc[b][t][0][1], inv), a.add[o]));
        double2 v1 = cfma(e0, acc[b][t][1][0], cfma(e1, acc[b][t][1][1], a.add[o + nL]));
        if (a.mid.tab) mid_apply(mid_op(a.mid, gg, nL, p, lam), v0, v1);
        a.out[o] = v0;
        a.out[o + nL] = v1;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Plan setup
// ---------------------------------------------------------------------------

// tab[g][0..2][p] = sum_s (v0 v0, v0 v1, v1 v1)[s] / (sigma_gs + lambda_p)
__global__ __launch_bounds__(256) void modal_table_kernel(const double2* sig, int64_t sS, int64_t sG, int nS, int nG,
                                                          int nL, const double2* lam, const double2* lamlo,
                                                          const double2* v0, const double2* v1, double2* tab) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)nG * nL) return;
  const int64_t g = i / nL;
  const int p = (int)(i - g * nL);
  double2 t00 = make_double2(0, 0), t01 = t00, t11 = t00;
  for (int s = 0; s < nS; ++s) {
    const double2 D = crcp(cadd(cadd(sig[s * sS + g * sG], lam[p]), lamlo[p]));
    const double2 x = cmul(v0[s], D);
    t00 = cfma(v0[s], x, t00);
    t01 = cfma(v1[s], x, t01);
    t11 = cfma(v1[s], cmul(v1[s], D), t11);
  }
  tab[g * 3 * nL + p] = t00;
  tab[(g * 3 + 1) * nL + p] = t01;
  tab[(g * 3 + 2) * nL + p] = t11;
}

// MV = M V for the mass matrix of an axis (V [n][n], rows i), and its transpose
__global__ __launch_bounds__(256) void mass_vec_kernel(const double2* __restrict__ V, int n, double h,
                                                       double2* __restrict__ MV, double2* __restrict__ MVT) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)n * n) return;
  const int i = (int)(e / n), p = (int)(e - (int64_t)i * n);
  const double d = (i == 0 || i == n - 1 ? 2.0 : 4.0) * h / 6.0;
  double2 v = cscale(V[e], d);
  if (i > 0) v = cadd(v, cscale(V[e - n], h / 6.0));
  if (i < n - 1) v = cadd(v, cscale(V[e + n], h / 6.0));
  if (MV) MV[e] = v;
  if (MVT) MVT[(int64_t)p * n + i] = v;
}

__global__ __launch_bounds__(256) void transpose_kernel(const double2* __restrict__ in, int n, double2* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)n * n) return;
  const int64_t i = e / n, p = e - i * n;
  out[p * n + i] = in[e];
}

// nrm[p] = h sum_i |V[i][p]|^2
__global__ __launch_bounds__(256) void col_norms_kernel(const double2* __restrict__ V, int n, double h, double* nrm) {
  const int p = (int)blockIdx.x * 256 + threadIdx.x;
  if (p >= n) return;
  double s = 0;
  for (int i = 0; i < n; ++i) {
    const double2 v = V[(int64_t)i * n + p];
    s += v.x * v.x + v.y * v.y;
  }
  nrm[p] = s * h;
}

unsigned blocks_of(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_modal_gather(const double2* p0, int64_t g0, int nt0, double2* o0, const double2* p1, int64_t g1,
                               int nt1, double2* o1, int nL, const int* skip, hipStream_t s) {
  const int64_t blocks = (g0 + g1) * ((2 * nL + 63) / 64);
  if (blocks < 1 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(modal_gather_kernel, dim3((unsigned)blocks), dim3(64 * kGatherWaves), 0, s, p0, g0, nt0, o0, p1,
                     nt1, o1, nL, skip);
  return hipGetLastError();
}

hipError_t launch_modal_rows(const double2* Q, int nL, int nb, const ModalRows* sets, int nsets, const int* skip,
                             hipStream_t s) {
  if (!Q || nL < 1 || nb < 1 || nsets < 1 || nsets > 2) return hipErrorInvalidValue;
  ModalRows s1;
  s1.n = 0;
  if (nsets > 1) s1 = sets[1];
  auto tiles = [&](int n, int64_t b) { return (2 * (int64_t)nb * n + b - 1) / b; };
  auto blocks = [&](int64_t b) { return (tiles(sets[0].n, b) + tiles(s1.n, b)) * ((nL + b - 1) / b); };
  if (blocks(32) > 0x7fffffffLL) return hipErrorInvalidValue;
  if (cgemm_tile(blocks(64)) == 1)
    hipLaunchKernelGGL(modal_rows_kernel<1>, dim3((unsigned)blocks(32)), dim3(256), 0, s, Q, nL, nb, sets[0], s1,
                       (int)tiles(sets[0].n, 32), skip);
  else
    hipLaunchKernelGGL(modal_rows_kernel<2>, dim3((unsigned)blocks(64)), dim3(256), 0, s, Q, nL, nb, sets[0], s1,
                       (int)tiles(sets[0].n, 64), skip);
  return hipGetLastError();
}

hipError_t launch_modal_mid(const ModalMid& m, int nb, int nG, int nL, const double2* lam, const double2* in,
                            double2* out, const int* skip, hipStream_t s) {
  const int64_t n = (int64_t)nb * nG * nL;
  if (n < 1 || (n + 255) / 256 > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(modal_mid_kernel, dim3(blocks_of(n)), dim3(256), 0, s, m, nb, nG, nL, lam, in, out, skip);
  return hipGetLastError();
}

hipError_t launch_modal_sum(const ModalSum& a, hipStream_t s) {
  if (a.nb < 1 || a.nS < 2 || a.nG < 2 || a.nL < 1) return hipErrorInvalidValue;
  auto blocks = [&](int tg, int nbt) {
    return (int64_t)((a.nL + 63) / 64) * ((a.nG / 2 + tg) / tg) * ((a.nb + nbt - 1) / nbt);
  };
  const dim3 t(64 * kSumWaves);
  // the larger tiles while they fill the chip (two blocks per compute unit)
  if (a.nb > 1 && blocks(2, 2) >= 512) {
    if (blocks(2, 2) > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((modal_sum_kernel<2, 2>), dim3((unsigned)blocks(2, 2)), t, 0, s, a);
  } else if (blocks(4, 1) >= 512) {
    hipLaunchKernelGGL((modal_sum_kernel<4, 1>), dim3((unsigned)blocks(4, 1)), t, 0, s, a);
  } else if (blocks(2, 1) >= 512) {
    hipLaunchKernelGGL((modal_sum_kernel<2, 1>), dim3((unsigned)blocks(2, 1)), t, 0, s, a);
  } else {
    hipLaunchKernelGGL((modal_sum_kernel<1, 1>), dim3((unsigned)blocks(1, 1)), t, 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_modal_table(const double2* sig, int64_t sS, int64_t sG, int nS, int nG, int nL, const double2* lam,
                              const double2* lamlo, const double2* v0, const double2* v1, double2* tab,
                              hipStream_t s) {
  hipLaunchKernelGGL(modal_table_kernel, dim3(blocks_of((int64_t)nG * nL)), dim3(256), 0, s, sig, sS, sG, nS, nG, nL,
                     lam, lamlo, v0, v1, tab);
  return hipGetLastError();
}

hipError_t launch_mass_vec(const double2* V, int n, double h, double2* MV, double2* MVT, hipStream_t s) {
  hipLaunchKernelGGL(mass_vec_kernel, dim3(blocks_of((int64_t)n * n)), dim3(256), 0, s, V, n, h, MV, MVT);
  return hipGetLastError();
}

hipError_t launch_transpose(const double2* in, int n, double2* out, hipStream_t s) {
  hipLaunchKernelGGL(transpose_kernel, dim3(blocks_of((int64_t)n * n)), dim3(256), 0, s, in, n, out);
  return hipGetLastError();
}

hipError_t launch_col_norms(const double2* V, int n, double h, double* nrm, hipStream_t s) {
  hipLaunchKernelGGL(col_norms_kernel, dim3(blocks_of(n)), dim3(256), 0, s, V, n, h, nrm);
  return hipGetLastError();
}

}  // namespace helm
