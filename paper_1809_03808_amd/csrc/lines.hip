// Batched tridiagonal solves: geometry, factor tables and launches (the kernels
// are in lines_kernel.h).
#include "dd.h"
#include "lines_kernel.h"

namespace helm {

namespace linek {
extern template hipError_t launch_lines_kernel<double2, true, true>(const LineDev&, int, int64_t, hipStream_t);
extern template hipError_t launch_lines_kernel<double2, true, false>(const LineDev&, int, int64_t, hipStream_t);
extern template hipError_t launch_lines_kernel<double2, false, true>(const LineDev&, int, int64_t, hipStream_t);
extern template hipError_t launch_lines_kernel<double2, false, false>(const LineDev&, int, int64_t, hipStream_t);
extern template hipError_t launch_lines_kernel<float2, true, true>(const LineDev&, int, int64_t, hipStream_t);
extern template hipError_t launch_lines_kernel<float2, true, false>(const LineDev&, int, int64_t, hipStream_t);
extern template hipError_t launch_lines_kernel<float2, false, true>(const LineDev&, int, int64_t, hipStream_t);
extern template hipError_t launch_lines_kernel<float2, false, false>(const LineDev&, int, int64_t, hipStream_t);
}  // namespace linek

namespace {

using namespace linek;

// 1/a: a reciprocal with one Newton step in double-double (by long division the
// factor table of 4096^2 took 3.5 ms a family, so 1.8).
__device__ inline cdd cdd_rcp(cdd a) {
  const dd den = dd_add(dd_mul(a.re, a.re), dd_mul(a.im, a.im));
  const double r0 = rcp_nr(den.hi);
  const dd r = dd_add(dd_of(r0), dd_mul_d(dd_sub(dd_of(1.0), dd_mul_d(den, r0)), r0));
  return {dd_mul(a.re, r), dd_neg(dd_mul(a.im, r))};
}

// Factor table: for every line matrix (l, m) and lane chunk q, the reciprocal
// pivot entering the chunk of the Thomas elimination, 1/p_x = 1 / (d_x - e^2 / p_{x-1})
// over the rows before it.  One thread per line, once per plan, in double-double
// arithmetic on the coefficients that the solves round: an entering pivot that
// differs from the one that the rows before it end with changes the matrix at
// that chunk boundary, so the rounding errors gathered over all rows must not
// reach the table.  (Composed in FP64 as 2 x 2 Moebius maps in a scan over the
// chunks, they were most of the residual of a plain FP64 solve: 256^3 at 10 points
// per wavelength 7.0e-11 with line sweeps and 7.4e-11 with the boundary steps in the
// eigenbasis, which does not share them, now 6.2e-13 and 1.3e-13; 512^3 1.3e-10, now
// 2.0e-12; 4096^2 3.1e-9, now 4.5e-11, and 5.6e-11 with the recurrence in FP64.)
__global__ __launch_bounds__(64) void factor_kernel(LineDev a, int P, int64_t lines, double2* piv) {
  const int64_t line = (int64_t)blockIdx.x * 64 + threadIdx.x;  // l * nI + m
  if (line >= lines) return;
  const RowCoef rc = coef_of_sigma(a, line_sigma(a, line / a.nI, line % a.nI));
  double2* out = piv + line * P;
  out[0] = make_double2(0, 0);
  const cdd e2 = cdd_of(rc.off2);
  cdd ip = cdd_zero();
  int x = 0;
  for (int q = 1; q < P; ++q) {
    for (const int end = chunk_start(q, a.c, a.r); x < end; ++x)
      ip = cdd_rcp(cdd_sub(cdd_of(x == 0 ? rc.dlo : rc.dint), cdd_mul(e2, ip)));
    out[q] = make_double2(ip.re.hi, ip.im.hi);
  }
}

LineDev make_dev(const LineArgs& a, int P, int c) {
  LineDev d;
  d.nb = a.nb; d.nO = a.nO; d.nI = a.nI; d.nL = a.nL; d.c = c; d.r = a.nL - P * (c - 1) < P ? a.nL - P * (c - 1) : P; d.red = a.red;
  d.sO = a.sO; d.sI = a.sI; d.sC = a.sC;
  d.hL = a.hL;
  d.m_end = 2.0 * a.hL / 6.0;
  d.m_int = 4.0 * a.hL / 6.0;
  d.m_off = a.hL / 6.0;
  d.k_off = -1.0 / a.hL;
  d.kLo = a.kLo; d.kHi = a.kHi;
  d.in = a.in;
  d.alpha0 = a.alpha0; d.alpha1 = a.alpha1; d.PO = a.PO;
  d.beta0 = a.beta0; d.beta1 = a.beta1; d.PI = a.PI;
  d.rho0 = a.rho0; d.rho1 = a.rho1;
  d.piv = a.piv;
  d.sTab = a.sTab;
  d.out = a.out; d.part = a.part;
  d.skip = a.skip;
  d.tile = d.ntiles = d.iters = 0;
  d.tl = d.tm = 0;
  d.xcd = 0;
  return d;
}

}  // namespace

// The smallest power-of-two P with 8 P >= nL, and balanced chunks of c =
// ceil(nL / P) or c - 1 rows; lines of P * 8 + 1 rows with P >= 64 (the 2^k + 1
// node counts from 513 up) P lanes of 8 rows plus the extra row of the last
// lane.  (Below 64 lanes the extra-row variant of the reducing kernel would drop
// to one wave per SIMD.)
void lines_geometry(int nL, int* P, int* c, int* NT) {
  int p = 1;
  while (p * 8 < nL) p <<= 1;
  if (p >= 128 && nL == p * 4 + 1) p >>= 1;
  *P = p;
  *c = nL == p * 8 + 1 ? 8 : (p == 1 && nL < 4 ? 4 : (nL + p - 1) / p);
  *NT = p > 256 ? p : 256;
}

hipError_t launch_line_factors(const LineArgs& a, double2* piv, hipStream_t s) {
  int P, c, NT;
  lines_geometry(a.nL, &P, &c, &NT);
  if (a.nL < 3 || P > 512) return hipErrorInvalidValue;
  const LineDev d = make_dev(a, P, c);
  const int64_t lines = (int64_t)a.nO * a.nI;
  if (lines <= 0) return hipSuccess;
  hipLaunchKernelGGL(factor_kernel, dim3((unsigned)((lines + 63) / 64)), dim3(64), 0, s, d, P, lines, piv);
  return hipGetLastError();
}

hipError_t launch_lines(LineArgs a, hipStream_t s) {
  if (a.nL < 3 || !a.piv) return hipErrorInvalidValue;
  if ((int64_t)a.nb * a.nO * a.nI + a.tile >= 0x7fffffffLL) return hipErrorInvalidValue;
  int P, c, NT;
  lines_geometry(a.nL, &P, &c, &NT);
  if (P > 512) return hipErrorInvalidValue;
  LineDev d = make_dev(a, P, c);
  const int LPB = NT / P;
  int64_t blocks;
  if (a.red == 1 || a.red == 2 || a.red == 3) {
    const int64_t extent = a.red == 1 ? a.nI : a.nO;
    const int64_t groups = a.red == 1   ? (int64_t)a.nb * a.nO
                           : a.red == 2 ? (int64_t)a.nb * a.nI
                                        : (int64_t)a.nb * ((a.nI + LPB - 1) / LPB);
    d.tile = a.tile;
    d.ntiles = (int)((extent + a.tile - 1) / a.tile);
    if (d.ntiles != a.ntiles) return hipErrorInvalidValue;
    blocks = groups * d.ntiles;
  } else if (a.tile_m > 0) {
    // storing launches over (outer, inner) mode tiles: the rank-2 rows of an
    // inner mode (PO) are then read again only once per outer tile, those of
    // an outer mode (PI) once per inner tile
    if (a.tile_l < 1 || (a.tile_m & (a.tile_m - 1))) return hipErrorInvalidValue;
    d.tl = a.tile_l;
    d.tm = a.tile_m;
    d.tile = a.tile_l * a.tile_m;
    const int64_t nt = (int64_t)a.nb * ((a.nO + a.tile_l - 1) / a.tile_l) * ((a.nI + a.tile_m - 1) / a.tile_m);
    if (nt > 0x7fffffffLL) return hipErrorInvalidValue;
    d.ntiles = (int)nt;
    d.xcd = nt % 8 == 0 ? 1 : 0;
    blocks = nt;
  } else {
    const int64_t lines = (int64_t)a.nb * a.nO * a.nI;
    d.tile = a.tile;
    d.ntiles = (int)((lines + a.tile - 1) / a.tile);
    blocks = d.ntiles;
  }
  if (a.red == 3) {
    d.iters = d.tile;  // one l per iteration, the slots take LPB consecutive m
  } else {
    if (d.tile % LPB) return hipErrorInvalidValue;
    d.iters = d.tile / LPB;
  }
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  // one storage kind for the input and output lines and the rank-2 rows
  if ((a.in && a.out && a.in_kind != a.out_kind)) return hipErrorInvalidValue;
  const int kind = a.in ? a.in_kind : a.out_kind;
  if ((a.PO || a.PI) && a.r2_kind != kind) return hipErrorInvalidValue;
  // the SPEC kernels' conditions
  const bool spec = a.real_sigma && (a.red ? a.in && !a.PO && !a.PI : a.PO || a.PI);
  auto go = [&](auto t, auto sp) {
    using T = decltype(t);
    constexpr bool S = decltype(sp)::value;
    return d.red ? linek::launch_lines_kernel<T, true, S>(d, P, blocks, s)
                 : linek::launch_lines_kernel<T, false, S>(d, P, blocks, s);
  };
  using std::false_type;
  using std::true_type;
  if (kind == ST_C64) return spec ? go(float2{}, true_type{}) : go(float2{}, false_type{});
  return spec ? go(double2{}, true_type{}) : go(double2{}, false_type{});
}

}  // namespace helm
