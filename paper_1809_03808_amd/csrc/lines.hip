// Batched tridiagonal solves: geometry, factor tables and launches (the kernels
// are in lines_kernel.h).
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

// Factor table: for every line matrix (l, m) and lane chunk q, the reciprocal
// pivot entering the chunk of the Thomas elimination.  Lane q
// composes the Moebius maps of its rows and a scan over the lanes gives the
// pivot state entering each chunk.  Runs once per plan; one block of P lanes
// per line.  The solves regenerate the pivots inside each chunk from it.
__global__ void factor_kernel(LineDev a, int P, double2* piv) {
  extern __shared__ double smem_d[];
  Mob* buf = reinterpret_cast<Mob*>(smem_d);
  const int q = threadIdx.x;
  const int64_t line = blockIdx.x;  // l * nI + m
  const int64_t l = line / a.nI, m = line % a.nI;
  const RowCoef rc = row_coef(a, l, m);
  const int x0 = chunk_start(q, a.c, a.r), rows = q < a.r ? a.c : a.c - 1;
  Mob G;
  G.a = make_double2(1, 0); G.b = make_double2(0, 0);
  G.c = make_double2(0, 0); G.d = make_double2(1, 0);
  for (int j = 0; j < rows; ++j) {
    const int x = x0 + j;
    const double2 dg = diag_of(rc, x, a.nL);
    const double2 e2 = has_e(x, a.nL) ? rc.off2 : make_double2(0, 0);
    Mob n;
    n.a = csub(cmul(dg, G.a), cmul(e2, G.c));
    n.b = csub(cmul(dg, G.b), cmul(e2, G.d));
    n.c = G.a;
    n.d = G.b;
    G = n;
  }
  mob_norm(G);
  // Hillis-Steele inclusive scan (later * earlier), then shift.
  buf[q] = G;
  __syncthreads();
  for (int d = 1; d < P; d <<= 1) {
    Mob mine = buf[q];
    Mob other = q >= d ? buf[q - d] : mine;
    __syncthreads();
    if (q >= d) {
      mine = mob_mul(mine, other);
      mob_norm(mine);
      buf[q] = mine;
    }
    __syncthreads();
  }
  double2 ip = make_double2(0, 0);
  if (q > 0) {
    const Mob E = buf[q - 1];
    // state entering the chunk: E (1, 0)^T = (E.a, E.c), 1/p = E.c / E.a
    ip = cmul(E.c, crcp(E.a));
  }
  piv[line * P + q] = ip;
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
  hipLaunchKernelGGL(factor_kernel, dim3((unsigned)lines), dim3(P), (size_t)P * sizeof(Mob), s, d, P, piv);
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
