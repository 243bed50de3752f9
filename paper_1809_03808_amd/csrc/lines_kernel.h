// Batched complex tridiagonal solves along the last axis.
//
// Every mode of the periodised axes leaves one tridiagonal system along the
// last axis: for the 2D blocks of H_B and H_A (eqs. (HB2D), (HA2D), Section
// 4.1.2) T = (lambda - w^2) M_2 + K_2, and in 3D, after the inner transform in
// x_2, T = (lambda_1 + lambda_2 - w^2) M_3 + K_3 (eqs. (HA3D), (HB3D), (A2D2),
// (B2D2)).  The matrices depend on the mode only through sigma, so nothing is
// stored: coefficients are regenerated per row.
//
// Elimination order.  The elimination is exactly the sequential Thomas
// algorithm (LU without pivoting, pivots p_x = d_x - e_x^2 / p_{x-1}).  With an
// absorbing face at x = 0 the first pivot has a negative imaginary part and,
// for real sigma, the map p -> d - e^2/p keeps it there, so no pivot vanishes.
// A partitioned (SPIKE-type) elimination would instead factor Dirichlet
// sub-blocks of the line, which are real and indefinite and can be singular
// for some sigma; it is not used.
//
// Parallelism.  A line of nL rows is owned by P lanes (P a power of two, one
// wave or a few), lane q holding the rows [q c, q c + c).  The substitutions of
// Thomas are associative and are evaluated by exclusive scans across the P
// lanes:
//   forward  z_x = d_x - e_x / p_{x-1} z_{x-1}          affine maps z -> F z + G
//   backward y_x = (z_x - e_{x+1} y_{x+1}) / p_x       affine maps, reversed
// Each lane composes its c rows, the scan supplies the state entering the
// chunk, and the lane then re-runs its rows sequentially.  The pivots depend on
// sigma only: the reciprocal pivot entering each chunk is computed once per plan
// (factor_kernel, row after row; the paper likewise factors the line matrices
// at initialisation), and a solve regenerates the c pivots of its chunk from it
// (c divisions instead of c table reads).  Moves between lanes are register moves
// inside a wave and one LDS exchange between the waves of a line.
// Arithmetic is FP64 whatever the storage precision.
//
// Right-hand sides may be generated from boundary planes (the rank-2 terms of
// Steps 2 and 3, eqs. (step2-1), (step3term)), and solutions may be reduced
// with per-mode weights into boundary partial sums (eqs. (2dBs1), (step2-3)),
// so the intermediate solutions z_1, z_2 never reach memory.
#pragma once

#include "helm_internal.h"

namespace helm {

namespace linek {

struct Aff {  // z -> f z + g
  double2 f, g;
};

__device__ inline Aff aff_then(const Aff& later, const Aff& earlier) {  // later o earlier
  Aff o;
  o.f = cmul(later.f, earlier.f);
  o.g = cfma(later.f, earlier.g, later.g);
  return o;
}

__device__ inline Aff aff_ident() {
  Aff a;
  a.f = make_double2(1, 0);
  a.g = make_double2(0, 0);
  return a;
}

__device__ inline double2 shfl_up2(double2 v, int d, int w) {
  return make_double2(__shfl_up(v.x, d, w), __shfl_up(v.y, d, w));
}
__device__ inline double2 shfl_down2(double2 v, int d, int w) {
  return make_double2(__shfl_down(v.x, d, w), __shfl_down(v.y, d, w));
}
__device__ inline Aff shfl_up_aff(const Aff& a, int d, int w) {
  Aff o;
  o.f = shfl_up2(a.f, d, w);
  o.g = shfl_up2(a.g, d, w);
  return o;
}
__device__ inline Aff shfl_down_aff(const Aff& a, int d, int w) {
  Aff o;
  o.f = shfl_down2(a.f, d, w);
  o.g = shfl_down2(a.g, d, w);
  return o;
}

// Moves of a 64-bit value across lanes with the data-parallel primitives:
// lanes whose source lane is outside the pattern (or whose row is masked
// off) keep `old`.
template <int CTRL, int ROWMASK>
__device__ inline double dpp_d(double src, double old) {
  const unsigned long long s = __builtin_bit_cast(unsigned long long, src);
  const unsigned long long o = __builtin_bit_cast(unsigned long long, old);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)o, (int)(unsigned)s, CTRL, ROWMASK, 0xF, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)(o >> 32), (int)(unsigned)(s >> 32), CTRL,
                                                            ROWMASK, 0xF, false);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Same with every row enabled and zero where no source lane exists
// (bound_ctrl), which needs no initialised destination.
template <int CTRL>
__device__ inline double dpp_d0(double src) {
  const unsigned long long s = __builtin_bit_cast(unsigned long long, src);
  const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)s, CTRL, 0xF, 0xF, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(s >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
template <int CTRL, int ROWMASK = 0xF>
__device__ inline Aff dpp_aff(const Aff& v) {  // identity where nothing arrives
  Aff o;
  o.f.x = dpp_d<CTRL, ROWMASK>(v.f.x, 1.0);
  if constexpr (ROWMASK == 0xF) {
    o.f.y = dpp_d0<CTRL>(v.f.y);
    o.g.x = dpp_d0<CTRL>(v.g.x);
    o.g.y = dpp_d0<CTRL>(v.g.y);
  } else {
    o.f.y = dpp_d<CTRL, ROWMASK>(v.f.y, 0.0);
    o.g.x = dpp_d<CTRL, ROWMASK>(v.g.x, 0.0);
    o.g.y = dpp_d<CTRL, ROWMASK>(v.g.y, 0.0);
  }
  return o;
}
// DPP controls (GFX9 encoding): row_shl:n = 0x100 + n, row_shr:n = 0x110 + n,
// wave_shl:1 = 0x130, wave_shr:1 = 0x138, row_bcast:15 = 0x142, row_bcast:31 =
// 0x143, row_newbcast:0 = 0x150.
constexpr int kRowShl1 = 0x101, kRowShl2 = 0x102, kRowShl4 = 0x104, kRowShl8 = 0x108;
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143, kRowFirst = 0x150;
constexpr int kWaveShl1 = 0x130, kWaveShr1 = 0x138;

// Inclusive prefix composition within groups of W lanes (W = 16, 32 or 64;
// later lanes applied after earlier ones): four in-row steps, then the row
// broadcasts that carry row totals to the following rows.
template <int W>
__device__ inline Aff dpp_inclusive(Aff v) {
  v = aff_then(v, dpp_aff<kRowShr1>(v));
  v = aff_then(v, dpp_aff<kRowShr2>(v));
  v = aff_then(v, dpp_aff<kRowShr4>(v));
  v = aff_then(v, dpp_aff<kRowShr8>(v));
  if constexpr (W >= 32) v = aff_then(v, dpp_aff<kRowBcast15, 0xA>(v));
  if constexpr (W >= 64) v = aff_then(v, dpp_aff<kRowBcast31, 0xC>(v));
  return v;
}

// The value of the first lane of the following row (rows 0 and 2; rows 1 and 3
// get their own first lane's).
__device__ inline double next_row_first(double v) {
  const unsigned long long s = __builtin_bit_cast(unsigned long long, v);
  unsigned w[2] = {(unsigned)s, (unsigned)(s >> 32)};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const unsigned f = (unsigned)__builtin_amdgcn_mov_dpp((int)w[i], kRowFirst, 0xF, 0xF, true);
    // swaps the odd rows of the first operand with the even rows of the second
    w[i] = __builtin_amdgcn_permlane16_swap(f, f, false, false)[1];
  }
  return __builtin_bit_cast(double, ((unsigned long long)w[1] << 32) | w[0]);
}
__device__ inline double lane_value(double v, int l) {  // wave-uniform
  const unsigned long long s = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)s, l);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(s >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Inclusive suffix composition (earlier lanes applied after later ones): the
// row shifts run the other way; the total of a row is in its first lane, which
// no row broadcast carries backwards, so rows 0 and 2 take that of rows 1 and 3
// through a swap of rows and the lower half of the wave that of the upper half
// through scalar registers.
template <int W>
__device__ inline Aff dpp_inclusive_rev(Aff v) {
  v = aff_then(v, dpp_aff<kRowShl1>(v));
  v = aff_then(v, dpp_aff<kRowShl2>(v));
  v = aff_then(v, dpp_aff<kRowShl4>(v));
  v = aff_then(v, dpp_aff<kRowShl8>(v));
  const int lane = threadIdx.x & 63;
  if constexpr (W >= 32) {
    Aff o;
    o.f = make_double2(next_row_first(v.f.x), next_row_first(v.f.y));
    o.g = make_double2(next_row_first(v.g.x), next_row_first(v.g.y));
    if (!(lane & 16)) v = aff_then(v, o);
  }
  if constexpr (W >= 64) {
    Aff o;
    o.f = make_double2(lane_value(v.f.x, 32), lane_value(v.f.y, 32));
    o.g = make_double2(lane_value(v.g.x, 32), lane_value(v.g.y, 32));
    if (!(lane & 32)) v = aff_then(v, o);
  }
  return v;
}

// Exclusive scans of affine maps over the P lanes of a line (lanes
// [slot*P, slot*P + P) of the block).  Forward: lane q receives
// A_{q-1} o ... o A_0; backward: lane q receives A_{q+1} o ... o A_{P-1}.
// Lines of 16 lanes and more scan with moves between registers, shorter ones
// with shuffles.  (A shuffle is an LDS instruction: with shuffles at 16 and 32
// lanes, and the backward scan of 64 lanes made a prefix scan by two reversals
// through them, they were 96 of the 166 LDS instructions of a storing wave at
// 256^3 FP64, and each scan six dependent LDS round trips.)
// For P > 64 the waves of a line exchange their totals through LDS (`wbuf`,
// NT/64 entries; forward and backward scans use different buffers, so one
// barrier per scan suffices: the next write to a buffer follows the other
// scan's barrier).  Every thread of the block must call these.
template <int P>
__device__ inline Aff scan_fwd(Aff v, int q, Aff* wbuf) {
  constexpr int W = P < 64 ? P : 64;
  Aff ex;
  if constexpr (W >= 16) {
    v = dpp_inclusive<W>(v);
    ex = dpp_aff<W == 16 ? kRowShr1 : kWaveShr1>(v);
    if (W == 32 && q == 0) ex = aff_ident();  // else the other line's last lane
  } else {
    const int lq = q & (W - 1);
#pragma unroll
    for (int d = 1; d < W; d <<= 1) {
      const Aff o = shfl_up_aff(v, d, W);
      if (lq >= d) v = aff_then(v, o);
    }
    ex = shfl_up_aff(v, 1, W);
    if (lq == 0) ex = aff_ident();
  }
  if constexpr (P > 64) {
    const int wv = threadIdx.x >> 6;          // wave in block
    const int w0 = wv - (q >> 6);             // first wave of this line
    if ((q & 63) == 63) wbuf[wv] = v;         // inclusive wave total
    __syncthreads();
    Aff pre = aff_ident();
    for (int w = w0; w < wv; ++w) pre = aff_then(wbuf[w], pre);
    ex = aff_then(ex, pre);
  }
  return ex;
}

template <int P>
__device__ inline Aff scan_bwd(Aff v, int q, Aff* wbuf) {
  constexpr int W = P < 64 ? P : 64;
  Aff ex;
  if constexpr (W >= 16) {
    v = dpp_inclusive_rev<W>(v);
    ex = dpp_aff<W == 16 ? kRowShl1 : kWaveShl1>(v);
    if (W == 32 && q == P - 1) ex = aff_ident();
  } else {
    const int lq = q & (W - 1);
#pragma unroll
    for (int d = 1; d < W; d <<= 1) {
      const Aff o = shfl_down_aff(v, d, W);
      if (lq + d < W) v = aff_then(v, o);
    }
    ex = shfl_down_aff(v, 1, W);
    if (lq == W - 1) ex = aff_ident();
  }
  if constexpr (P > 64) {
    const int wv = threadIdx.x >> 6;
    const int wl = wv - (q >> 6) + P / 64 - 1;       // last wave of this line
    if ((threadIdx.x & 63) == 0) wbuf[wv] = v;       // inclusive suffix total of the wave
    __syncthreads();
    Aff suf = aff_ident();
    for (int w = wl; w > wv; --w) suf = aff_then(wbuf[w], suf);
    ex = aff_then(ex, suf);
  }
  return ex;
}

struct LineDev {
  int nb, nO, nI, nL, c, r, red, tile, ntiles, iters;  // c, r: chunk rows and the lanes that own c (not c - 1) of them
  int tl, tm;  // red == 0 with tm > 0: blocks take tiles of tl outer x tm inner modes
  int xcd;     // with tiles: consecutive blocks of one XCD take consecutive tiles
  const double2* sO;
  const double2* sI;
  double2 sC;
  double hL, m_end, m_int, m_off, k_off;
  double2 kLo, kHi;
  const void* in;
  const double2 *alpha0, *alpha1, *beta0, *beta1, *rho0, *rho1;
  const void *PO, *PI;  // rank-2 rows, of the lines' storage type
  const double2* piv;   // [nO*nI][P]: reciprocal pivot entering the chunk of each lane
  const double2* sTab;  // [nO*nI] sigma per line, or null
  void* out;
  double2* part;
  const int* skip;
};

struct RowCoef {
  double2 dint, dlo, dhi, off, off2;
};

__device__ inline double2 line_sigma(const LineDev& a, int64_t l, int64_t m) {
  double2 sig;
  if (a.sTab) {
    sig = a.sTab[l * a.nI + m];
  } else {
    sig = a.sC;
    if (a.sO) sig = cadd(sig, a.sO[l]);
    if (a.sI) sig = cadd(sig, a.sI[m]);
  }
  return sig;
}
__device__ inline RowCoef coef_of_sigma(const LineDev& a, double2 sig) {
  RowCoef r;
  r.off = make_double2(sig.x * a.m_off + a.k_off, sig.y * a.m_off);  // sigma h/6 - 1/h
  r.off2 = cmul(r.off, r.off);
  r.dint = make_double2(sig.x * a.m_int + 2.0 / a.hL, sig.y * a.m_int);
  r.dlo = make_double2(sig.x * a.m_end + a.kLo.x / a.hL, sig.y * a.m_end + a.kLo.y / a.hL);
  r.dhi = make_double2(sig.x * a.m_end + a.kHi.x / a.hL, sig.y * a.m_end + a.kHi.y / a.hL);
  return r;
}

// First row of lane q: lanes below r own c rows, the others c - 1.
__host__ __device__ inline int chunk_start(int q, int c, int r) { return q * (c - 1) + (q < r ? q : r); }
// The lines of a block.  Line index (b, l, m) of slot `sl` at iteration `it`;
// false past the end of the tile's extent.  Line counts stay below 2^31 (checked
// at launch), so 32-bit index arithmetic suffices; the divisions (about thirty
// instructions each, against some four hundred of a whole 8-row chunk) are made
// once per block.  Reductions over l come in two layouts: red 2 gives a block
// one m and its slots consecutive l (lines nI nL elements apart); red 3 gives
// the slots of a block lpb consecutive m at one l per iteration, so one
// iteration reads lpb adjacent lines and the rows PI[b][l] once, and every slot
// keeps its own partial sum.  Storing launches take tiles of tl outer x tm inner
// modes (tm a power of two), or consecutive lines.
template <bool RED> struct BlockLines {
  uint32_t b, l, m;  // line of iteration 0, slot 0
  uint32_t first;    // consecutive storing launches: its index
  uint32_t tmsh;     // tiled ones: log2 tm

  __device__ BlockLines(const LineDev& a, uint32_t g, uint32_t t, uint32_t lpb) {
    const uint32_t nO = a.nO, nI = a.nI, base = t * (uint32_t)a.tile;
    first = tmsh = 0;
    if constexpr (RED) {
      if (a.red == 1) {         // g = b*nO + l
        b = g / nO;
        l = g - b * nO;
        m = base;
      } else if (a.red == 2) {  // g = b*nI + m
        b = g / nI;
        m = g - b * nI;
        l = base;
      } else {                  // g = b*nmg + mg, m = mg*lpb + sl
        const uint32_t nmg = (nI + lpb - 1) / lpb;
        b = g / nmg;
        m = (g - b * nmg) * lpb;
        l = base;
      }
    } else if (a.tm > 0) {      // t = (b, mt, lt)
      const uint32_t nlt = (nO + (uint32_t)a.tl - 1) / (uint32_t)a.tl;
      const uint32_t nmt = (nI + (uint32_t)a.tm - 1) / (uint32_t)a.tm;
      const uint32_t bm = t / nlt;
      b = bm / nmt;
      l = (t - bm * nlt) * (uint32_t)a.tl;
      m = (bm - b * nmt) * (uint32_t)a.tm;
      tmsh = 31u - (uint32_t)__builtin_clz((uint32_t)a.tm);
    } else {
      first = base;
      const uint32_t bl = base / nI;
      m = base - bl * nI;
      b = bl / nO;
      l = bl - b * nO;
    }
  }

  __device__ bool line(const LineDev& a, int lpb, int it, int sl, uint32_t& ob, uint32_t& ol, uint32_t& om) const {
    const uint32_t nO = a.nO, nI = a.nI, idx = (uint32_t)(it * lpb + sl);
    bool valid;
    ob = b;
    ol = l;
    om = m;
    if constexpr (RED) {
      if (a.red == 1) {
        om = m + idx;
        valid = om < nI;
      } else if (a.red == 2) {
        ol = l + idx;
        valid = ol < nO;
      } else {
        ol = l + (uint32_t)it;
        om = m + (uint32_t)sl;
        valid = ol < nO && om < nI;
      }
    } else if (a.tm > 0) {
      const uint32_t il = idx >> tmsh;
      ol = l + il;
      om = m + (idx - (il << tmsh));
      valid = idx < (uint32_t)a.tile && ol < nO && om < nI && b < (uint32_t)a.nb;
    } else {
      valid = first + idx < (uint32_t)a.nb * nO * nI;
      om = m + idx;
      if (om >= nI) {
        const uint32_t c = om / nI;
        om -= c * nI;
        ol = l + c;
        if (ol >= nO) {
          const uint32_t d = ol / nO;
          ol -= d * nO;
          ob = b + d;
        }
      }
    }
    if (!valid) ob = ol = om = 0;
    return valid;
  }
};

// Padded position of element e of a wave's staging area: one pad slot per 8
// elements, so that lanes reading rows lane*c + j (c = 8) hit distinct banks.
__device__ inline int stage_pos(int e) { return e + (e >> 3); }

// Memory layout and staging.  Line rows are contiguous in memory but lane q
// owns the contiguous chunk [q c, q c + c), so direct per-lane loads would
// touch 64 cache lines per wave instruction.  Instead every wave loads the
// rows of its lanes with consecutive lanes on consecutive rows (whole cache
// lines per instruction), assembles the right-hand side there, and passes the
// chunks through its own LDS area (72 c complex values, padded); solutions to
// be stored take the same route back.  Between the two, the area parks the
// lane's reciprocal pivots and then its backward multipliers.  A wave's area
// is only touched by that wave, whose LDS accesses execute in program order,
// except in the final cross-slot reduction, which is fenced by block
// barriers.
//
// EXACT lines have P * C rows, C for every lane (C = 8).  Then the only rows
// without a coupling to their predecessor / successor are x = 0 and x = nL - 1,
// and neither needs a guard: the entering reciprocal pivot of lane 0 is zero,
// which zeroes its first forward multiplier, and the last lane's backward
// recurrence starts from y = 0, which annihilates its last backward multiplier.
//
// BAL lines have any length in (P (C - 1), P C]: the first r = nL - P (C - 1)
// lanes own C rows and the others C - 1, so that no lane holds rows past the
// end of the line and only the last row of a chunk is conditional.  P is the
// smallest power of two with 8 P >= nL, hence C = 5 ... 8 (P = 1: 4 ... 8).
// Against chunks of 8 rows padded with identity rows and a guard at every row,
// a 129-row line does 160 rows' work instead of 256, with the loads batched as
// in the exact kernels.
//
// XR (with C = 8): the line has one row more, nL = P * 8 + 1 (the 2^k + 1
// node counts of the paper's grids).  The last lane owns it beside its chunk:
// it finishes the forward elimination through it after the forward scan
// (its pivot and value follow from the chunk's last ones), takes y_{nL-1},
// and folds it into its backward map, which becomes the constant map to the
// value entering its chunk from above.
// Storing launches are held to 128 registers where LDS admits four waves per
// SIMD and the kernel comes close: exact lines of 16 to 64 lanes, exact and
// balanced ones of 512.
//
// SPEC: sigma is real (the periodic branch of every periodised axis), so the
// off-diagonal entry and its square are (a complex product with them takes two
// instructions instead of four), and a reducing launch has an input and no
// rank-2 rows, and its first weight rho_0 is one real number (1/n).  These
// are the two reductions of a 3D solve in the eigenbasis, Step 1 in 2D and the
// storing launches of the fast method.
template <typename T, int NT, int P, int C, bool RED, bool XR, bool BAL, bool SPEC>
__global__ __launch_bounds__(NT, !RED && !XR && (NT == 512 || (!BAL && P >= 16 && P <= 64)) ? 4 : 1) void lines_kernel(LineDev a) {
  constexpr bool RANK2 = !(RED && SPEC);
  constexpr int NW = NT / 64;
  constexpr int PW = P < 64 ? P : 64;     // lanes of one line inside a wave
  constexpr int SPW = 64 / PW;            // lines per wave
  constexpr int LPB = NT / P;             // lines per block
  constexpr int NJ = (PW * C + 63) / 64;  // loads per lane that cover a wave's rows of one line
  __shared__ Aff wbuf[2][NW + 1];         // wave totals of the forward / backward scans
  extern __shared__ double2 stage[];      // NW areas of 72 c padded values
  if (a.skip && *a.skip) return;

  const int nL = BAL ? a.nL : P * C + (XR ? 1 : 0);
  const int nr = BAL ? a.r : P;           // lanes that own C rows
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // a line spans whole waves when P >= 64: its index is then wave-uniform
  const int slot = P >= 64 ? __builtin_amdgcn_readfirstlane(tid / P) : tid / P;
  const int q = tid - slot * P;
  const int x0 = BAL ? chunk_start(q, C, nr) : q * C;
  const bool full = !BAL || q < nr;       // this lane owns C rows, not C - 1
  const bool last = XR && q == P - 1;  // owner of the extra row
  const int wslot0 = (wv * 64) / P;                   // first line slot of this wave
  const int wq0 = P >= 64 ? (wv * 64) % P : 0;        // first lane of a line in this wave
  const int wx0 = BAL ? chunk_start(wq0, C, nr) : wq0 * C;  // first row this wave stages
  // rows of one line staged by this wave
  const int seg = BAL ? chunk_start(wq0 + PW, C, nr) - wx0 : PW * C;
  double2* S = stage + wv * (72 * C);
  const int sbase = P >= 64 ? x0 - wx0 : (lane / PW) * seg + x0;  // first staged element of this lane's chunk
  auto slot_of = [&](int j) { return stage_pos(sbase + j); };
  // row j of the chunk exists (only the last one may not)
  auto has_row = [&](int j) { return !BAL || j < C - 1 || full; };

  const uint32_t blk = blockIdx.x;
  uint32_t g = 0, t = 0;
  if (a.red) {
    g = blk / (uint32_t)a.ntiles;
    t = blk - g * (uint32_t)a.ntiles;
  } else if (a.xcd) {
    // blocks are dealt to the 8 XCDs in turn: block 8k + x takes tile
    // x ntiles/8 + k, so the blocks resident on one XCD work on
    // consecutive tiles (outer-mode tiles fastest), which share the rank-2
    // rows of their inner modes in that XCD's L2
    t = (blk & 7u) * ((uint32_t)a.ntiles >> 3) + (blk >> 3);
  } else {
    t = blk;
  }

  const BlockLines<RED> lines(a, g, t, LPB);

  double2 acc0[C], acc1[C];
  double2 accx0 = make_double2(0, 0), accx1 = accx0;  // the extra row (XR, last lane)
  if constexpr (RED) {
#pragma unroll
    for (int j = 0; j < C; ++j) acc0[j] = acc1[j] = make_double2(0, 0);
  }

  // Reducing launches without rank-2 rows (SPEC) load the next lines' rows,
  // sigma, entering pivots and weights into registers while the current lines
  // are solved: two waves per SIMD (the accumulators' registers) hide little of
  // a load's latency (against loads at the top of the iteration: 256^3 FP64
  // reductions 115 -> 73 us, 129^3 x 2 mixed 55 -> 37, 512^3 x 4 mixed 2.7 ->
  // 1.75 ms, 4096^2 FP64 132 -> 97 us).  FP64 chunks of 8 rows of uneven lines
  // and those with the extra row lack the registers; lines of fewer than 16
  // lanes would hold the rows of 8 lines and more.
  constexpr bool PREF = RED && SPEC && P >= 16 && (sizeof(T) == sizeof(float2) || !(XR || (BAL && C == 8)));
  T pre[PREF ? SPW * NJ : 1];
  double2 nsig = make_double2(0, 0), nip = nsig, nw1 = nsig;
  bool nvalid = false;
  // element of row r of the wave's part of a line; masked lanes read its first
  auto row_of = [&](int r) { return wx0 + (r < seg ? r : 0); };
  auto fetch = [&](int itn) {
#pragma unroll
    for (int si = 0; si < SPW; ++si) {
      uint32_t sb, sl, sm;
      lines.line(a, LPB, itn, wslot0 + si, sb, sl, sm);
      const T* in = reinterpret_cast<const T*>(a.in) + ((int64_t)(sb * a.nO + sl) * a.nI + sm) * nL;
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj) pre[si * NJ + jj] = in[row_of(jj * 64 + lane)];
    }
    uint32_t sb, sl, sm;
    nvalid = lines.line(a, LPB, itn, slot, sb, sl, sm);
    nsig = line_sigma(a, sl, sm);
    nip = q > 0 ? a.piv[(int64_t)(sl * a.nI + sm) * P + q] : make_double2(0, 0);
    nw1 = a.rho1[(a.red == 1) ? sm : sl];
  };
  if constexpr (PREF) {
    if (a.iters > 0) fetch(0);
  }

  for (int it = 0; it < a.iters; ++it) {
    const double2 psig = nsig, pip = nip, pw1 = nw1;
    const bool pvalid = nvalid;
    // ---- right-hand side, staged through LDS -------------------------------
    // A line past the end of the tile is read as line 0 and its results are
    // dropped.
    if constexpr (PREF) {
#pragma unroll
      for (int si = 0; si < SPW; ++si)
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
          const int r = jj * 64 + lane;
          if (r < seg) S[stage_pos(si * seg + r)] = to_d2(pre[si * NJ + jj]);
        }
      if (it + 1 < a.iters) fetch(it + 1);
    } else {
      // The input row and the four rank-2 rows of a batch of chunk rows (of SB
      // lines where a line has few) are loaded before any is used, combined in
      // registers and staged once.  Staged values updated source by source cost
      // five LDS accesses a row instead of one and a wait per source (storing
      // launches: 129^3 x 2 mixed 64 -> 41 us, 512^3 x 4 mixed 3.5 -> 3.06 ms,
      // 2049^2 FP64 51 -> 39 us, 4096^2 FP64 151 -> 139 us; batches of 8 rows
      // the same within 1%, with more registers).
      constexpr int NB0 = RED || P <= 64 ? 4 : 2;
      constexpr int NBAT = NB0 < NJ ? NB0 : NJ;
      constexpr int NU0 = !RED && sizeof(T) == sizeof(float2) ? 4 : 2;  // (registers)
      constexpr int SB = NU0 / NJ < 1 ? 1 : (NU0 / NJ < SPW ? NU0 / NJ : SPW);
      auto rhs = [&](auto has_in, auto has_po, auto has_pi) {
        constexpr bool HI = decltype(has_in)::value, HO = decltype(has_po)::value, HP = decltype(has_pi)::value;
#pragma unroll 1
        for (int si = 0; si < SPW; si += SB) {
          const T *in[SB], *po[SB], *pi[SB];
          double2 al0[SB], al1[SB], be0[SB], be1[SB];
#pragma unroll
          for (int k = 0; k < SB; ++k) {
            uint32_t sb, sl, sm;
            lines.line(a, LPB, it, wslot0 + si + k, sb, sl, sm);
            in[k] = reinterpret_cast<const T*>(a.in) + ((int64_t)(sb * a.nO + sl) * a.nI + sm) * nL;
            po[k] = reinterpret_cast<const T*>(a.PO) + (int64_t)(sb * 2) * a.nI * nL + (int64_t)sm * nL;
            pi[k] = reinterpret_cast<const T*>(a.PI) + (int64_t)((sb * a.nO + sl) * 2) * nL;
            if constexpr (HO) { al0[k] = a.alpha0[sl]; al1[k] = a.alpha1[sl]; }
            if constexpr (HP) { be0[k] = a.beta0[sm]; be1[k] = a.beta1[sm]; }
          }
#pragma unroll
          for (int j0 = 0; j0 < NJ; j0 += NBAT) {
            constexpr int NU = SB * NBAT;
            T v[NU], p0[NU], p1[NU], p2[NU], p3[NU];
#pragma unroll
            for (int u = 0; u < NU; ++u) {
              const int k = u / NBAT, j = j0 + u % NBAT;
              if (j >= NJ) continue;
              const int x = row_of(j * 64 + lane);
              if constexpr (HI) v[u] = in[k][x];
              if constexpr (HO) { p0[u] = po[k][x]; p1[u] = po[k][(int64_t)a.nI * nL + x]; }
              if constexpr (HP) { p2[u] = pi[k][x]; p3[u] = pi[k][nL + x]; }
            }
#pragma unroll
            for (int u = 0; u < NU; ++u) {
              const int k = u / NBAT, j = j0 + u % NBAT;
              if (j >= NJ) continue;
              const int r = j * 64 + lane;
              double2 d = make_double2(0, 0);
              if constexpr (HI) d = to_d2(v[u]);
              if constexpr (HO) d = cfma(al1[k], to_d2(p1[u]), cfma(al0[k], to_d2(p0[u]), d));
              if constexpr (HP) d = cfma(be1[k], to_d2(p3[u]), cfma(be0[k], to_d2(p2[u]), d));
              if (r < seg) S[stage_pos((si + k) * seg + r)] = d;
            }
            // the next batch's loads stay behind this one's registers
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      };
      using std::false_type;
      using std::true_type;
      // one branch per set of sources: loads under a condition each are
      // converted inside it and waited for one by one (512^3 x 4 mixed 4.4 ms)
      const bool hi = a.in, ho = RANK2 && a.PO, hp = RANK2 && a.PI;
      if constexpr (!RANK2) {
        rhs(true_type{}, false_type{}, false_type{});
      } else if (hi) {
        if (ho && hp) rhs(true_type{}, true_type{}, true_type{});
        else if (ho) rhs(true_type{}, true_type{}, false_type{});
        else if (hp) rhs(true_type{}, false_type{}, true_type{});
        else rhs(true_type{}, false_type{}, false_type{});
      } else {
        if (ho && hp) rhs(false_type{}, true_type{}, true_type{});
        else if (ho) rhs(false_type{}, true_type{}, false_type{});
        else if (hp) rhs(false_type{}, false_type{}, true_type{});
        else rhs(false_type{}, false_type{}, false_type{});
      }
    }

    uint32_t b, l, m;
    bool valid;
    if constexpr (PREF && !XR) {
      b = l = m = 0;
      valid = pvalid;
    } else {
      valid = lines.line(a, LPB, it, slot, b, l, m);
    }
    const double2 sig = PREF ? psig : line_sigma(a, l, m);
    RowCoef rc = coef_of_sigma(a, sig);
    if (SPEC) rc.dint.y = 0.0;
    const double2 moff = make_double2(-rc.off.x, -rc.off.y);  // -e
    // -e v and d - e^2 v; e is real in SPEC launches
    auto mul_moff = [&](double2 v) { return SPEC ? cscale(v, moff.x) : cmul(moff, v); };
    auto sub_off2 = [&](double2 v, double2 d) {
      return SPEC ? make_double2(fma(-rc.off2.x, v.x, d.x), fma(-rc.off2.x, v.y, d.y)) : cfms(rc.off2, v, d);
    };
    double2 z[C];
#pragma unroll
    for (int j = 0; j < C; ++j) z[j] = has_row(j) ? S[slot_of(j)] : make_double2(0, 0);
    const int64_t loff = ((int64_t)(b * a.nO + l) * a.nI + m) * nL;  // this lane's line
    double2 xrhs = make_double2(0, 0);  // right-hand side of the extra row
    if (XR && last && valid) {
      const int x = nL - 1;
      if (a.in) xrhs = to_d2(reinterpret_cast<const T*>(a.in)[loff + x]);
      if (RANK2 && a.PO) {
        const T* po = reinterpret_cast<const T*>(a.PO) + (int64_t)(b * 2) * a.nI * nL + (int64_t)m * nL;
        xrhs = cfma(a.alpha0[l], to_d2(po[x]), xrhs);
        xrhs = cfma(a.alpha1[l], to_d2(po[(int64_t)a.nI * nL + x]), xrhs);
      }
      if (RANK2 && a.PI) {
        const T* pi = reinterpret_cast<const T*>(a.PI) + (int64_t)((b * a.nO + l) * 2) * nL;
        xrhs = cfma(a.beta0[m], to_d2(pi[x]), xrhs);
        xrhs = cfma(a.beta1[m], to_d2(pi[nL + x]), xrhs);
      }
    }

    // ---- 1. pivots and forward composition --------------------------------
    // Reciprocal pivots: the chunk's entering value from the plan's factor
    // table, then the Thomas recurrence p_x = d_x - e^2 / p_{x-1}.
    // Forward substitution z_x = f_x z_{x-1} + d_x, f_x = -e / p_{x-1}: the
    // lane composes its rows into one affine map.  With m_x = -e / p_x its
    // factor is m_in m_x0 ... m_{last-1} and that of the backward map below
    // m_x0 ... m_last, so the product R of the common ones is formed once.
    const double2 ip_in = PREF ? pip : (q > 0 ? a.piv[(int64_t)(l * a.nI + m) * P + q] : make_double2(0, 0));
    Aff A;
    double2 R = make_double2(1, 0);
    double2 ipp_last;  // 1/p of the chunk's last row
    {
      double2 ipp = ip_in;
#pragma unroll
      for (int j = 0; j < C; ++j) {
        if (has_row(j)) {
          const double2 f = mul_moff(ipp);
          if (j == 0) {
            A.g = z[0];
          } else {
            R = j == 1 ? f : cmul(f, R);
            A.g = cfma(f, A.g, z[j]);
          }
          const bool end = !XR && q == P - 1 && (j == C - 1 || (BAL && j == C - 2 && !full));
          double2 pv = (j == 0 && q == 0) ? rc.dlo : (end ? rc.dhi : rc.dint);
          pv = sub_off2(ipp, pv);  // ipp = 0 at x = 0
          ipp = crcp_fast(pv);
          S[slot_of(j)] = ipp;
        }
      }
      ipp_last = ipp;
      A.f = cmul(mul_moff(ip_in), R);
    }
    // (the parked values are read back: kept in registers across the scans,
    // 40 more, they cost an occupancy level or the prefetch)
    asm volatile("" ::: "memory");
    const Aff Ein = scan_fwd<P>(A, q, wbuf[0]);

    // ---- 2. forward values, scaled for the back substitution --------------
    // h_x = z_x / p_x; the lane's slots now take the backward multipliers
    // g_x = -e / p_x.
    double2 yx = make_double2(0, 0);  // y of the extra row (XR, last lane)
    {
      double2 zp = Ein.g;
      double2 mp = mul_moff(ip_in);
#pragma unroll
      for (int j = 0; j < C; ++j) {
        if (has_row(j)) {
          zp = cfma(mp, zp, z[j]);
          const double2 ipj = S[slot_of(j)];
          z[j] = cmul(zp, ipj);
          mp = mul_moff(ipj);
          S[slot_of(j)] = mp;
        }
      }
      if (XR && last) {
        // extra row: w = r + (-e / p_{nL-2}) w_{nL-2}, p = d_hi - e^2 / p_{nL-2}
        const double2 wx = cfma(mul_moff(ipp_last), zp, xrhs);
        yx = cmul(wx, crcp_fast(sub_off2(ipp_last, rc.dhi)));
      }
    }

    asm volatile("" ::: "memory");
    // ---- 3. back substitution y_x = g_x y_{x+1} + h_x: composition, scan ---
    Aff B;
    B.f = cmul(mul_moff(ipp_last), R);
    B.g = z[C - 1];
#pragma unroll
    for (int j = C - 2; j >= 0; --j) B.g = cfma(S[slot_of(j)], B.g, z[j]);
    if (XR && last) {  // the value above the chunk is known: a constant map
      B.g = cfma(B.f, yx, B.g);
      B.f = make_double2(0, 0);
    }
    asm volatile("" ::: "memory");
    const Aff Bin = scan_bwd<P>(B, q, wbuf[1]);
    {
      double2 ynext = (XR && last) ? yx : Bin.g;
#pragma unroll
      for (int j = C - 1; j >= 0; --j) {
        if (has_row(j)) {
          ynext = cfma(S[slot_of(j)], ynext, z[j]);
          z[j] = ynext;
        }
      }
    }

    // ---- 4. epilogue -------------------------------------------------------
    if (a.out) {
#pragma unroll
      for (int j = 0; j < C; ++j)
        if (has_row(j)) S[slot_of(j)] = z[j];
      T* o = reinterpret_cast<T*>(a.out);
#pragma unroll 4
      for (int si = 0; si < SPW; ++si) {
        uint32_t sb, sl, sm;
        const bool sv = lines.line(a, LPB, it, wslot0 + si, sb, sl, sm);
        const int64_t soff = ((int64_t)(sb * a.nO + sl) * a.nI + sm) * nL;
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
          const int r = jj * 64 + lane, x = wx0 + r;
          if (r < seg && sv) o[soff + x] = from_d2<T>(S[stage_pos(si * seg + r)]);
        }
      }
    }
    if (XR && a.out && last && valid) reinterpret_cast<T*>(a.out)[loff + nL - 1] = from_d2<T>(yx);
    if constexpr (RED) {
      if (valid) {
        const uint32_t wi = (a.red == 1) ? m : l;
        const double2 w0 = SPEC ? make_double2(0, 0) : a.rho0[wi], w1 = PREF ? pw1 : a.rho1[wi];
        if (XR && last) {
          accx0 = SPEC ? cadd(yx, accx0) : cfma(w0, yx, accx0);
          accx1 = cfma(w1, yx, accx1);
        }
#pragma unroll
        for (int j = 0; j < C; ++j) {  // (a missing row holds zero)
          acc0[j] = SPEC ? cadd(z[j], acc0[j]) : cfma(w0, z[j], acc0[j]);
          acc1[j] = cfma(w1, z[j], acc1[j]);
        }
      }
    }
  }

  // ---- cross-slot reduction (fixed slot order) and partial write -----------
  if constexpr (RED) {
    double2* outp = a.part + ((int64_t)g * a.ntiles + t) * 2 * nL;
    // SPEC: rho_0 is the same real number for every mode (1/n of a periodic
    // axis), applied here to the plain sums
    const double sc0 = SPEC ? a.rho0[0].x : 1.0;
    if constexpr (SPEC) {
#pragma unroll
      for (int j = 0; j < C; ++j) acc0[j] = cscale(acc0[j], sc0);
      accx0 = cscale(accx0, sc0);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < C; ++j)
        if (has_row(j)) S[slot_of(j)] = k ? acc1[j] : acc0[j];
      if constexpr (XR) S[lane * 9 + 8] = k ? accx1 : accx0;  // the lane's pad slot (C = 8)
      __syncthreads();
      // staged position of row x of line slot sl (every slot uses its waves' areas)
      auto staged = [&](int sl, int x) {
        if (XR && x == nL - 1) {
          const int owner = sl * P + P - 1;
          return (owner >> 6) * (72 * C) + (owner & 63) * 9 + 8;
        }
        if constexpr (P <= 64) return (sl / SPW) * (72 * C) + stage_pos((sl % SPW) * seg + x);
        const int qq = !BAL || x < nr * C ? x / C : nr + (x - nr * C) / (C - 1);
        const int w = qq >> 6;
        return (sl * (P / 64) + w) * (72 * C) + stage_pos(x - (BAL ? chunk_start(w * 64, C, nr) : w * 64 * C));
      };
      if (a.red == 3) {
        // one partial per slot: part[(b nI + m) ntiles + t][k][x], m = mg LPB + sl
        const uint32_t nmg = ((uint32_t)a.nI + LPB - 1) / LPB;
        const uint32_t b3 = g / nmg, m0 = (g - b3 * nmg) * LPB;
        for (int e = tid; e < LPB * nL; e += NT) {
          const int sl = e / nL, x = e - sl * nL;
          if (m0 + (uint32_t)sl >= (uint32_t)a.nI) continue;
          a.part[(((int64_t)b3 * a.nI + m0 + sl) * a.ntiles + t) * 2 * nL + (int64_t)k * nL + x] =
              stage[staged(sl, x)];
        }
        continue;
      }
      for (int x = tid; x < nL; x += NT) {
        double2 s = make_double2(0, 0);
        for (int sl = 0; sl < LPB; ++sl) s = cadd(s, stage[staged(sl, x)]);
        outp[(int64_t)k * nL + x] = s;
      }
    }
  }
}

template <typename T, int NT, int P, int C, bool RED, bool XR, bool BAL, bool SPEC>
hipError_t launch_R(const LineDev& d, int64_t blocks, hipStream_t s) {
  // staging areas: up to 72 KB at NT = 512, above the default dynamic LDS
  // limit, so raise the limit for this kernel once
  static bool attr = false;
  constexpr int lds = (NT / 64) * 72 * C * (int)sizeof(double2);
  if (!attr) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&lines_kernel<T, NT, P, C, RED, XR, BAL, SPEC>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr = true;
  }
  hipLaunchKernelGGL((lines_kernel<T, NT, P, C, RED, XR, BAL, SPEC>), dim3((unsigned)blocks), dim3(NT), lds, s, d);
  return hipGetLastError();
}

// The kernel of a geometry (lines_geometry): exact lines, lines with the extra
// row, or balanced chunks of c and c - 1 rows.
template <typename T, bool RED, bool SPEC, int NT, int P>
hipError_t launch_P(const LineDev& d, int64_t blocks, hipStream_t s) {
  if (d.nL == P * 8) return launch_R<T, NT, P, 8, RED, false, false, SPEC>(d, blocks, s);
  if constexpr (P >= 64) {
    if (d.nL == P * 8 + 1) return launch_R<T, NT, P, 8, RED, true, false, SPEC>(d, blocks, s);
  }
  if (d.r < 0 || d.r > P || d.nL != P * (d.c - 1) + d.r) return hipErrorInvalidValue;
  switch (d.c) {
    case 4:
      if constexpr (P == 1) return launch_R<T, NT, P, 4, RED, false, true, SPEC>(d, blocks, s);
      return hipErrorInvalidValue;
    case 5: return launch_R<T, NT, P, 5, RED, false, true, SPEC>(d, blocks, s);
    case 6: return launch_R<T, NT, P, 6, RED, false, true, SPEC>(d, blocks, s);
    case 7: return launch_R<T, NT, P, 7, RED, false, true, SPEC>(d, blocks, s);
    case 8: return launch_R<T, NT, P, 8, RED, false, true, SPEC>(d, blocks, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, bool RED, bool SPEC>
hipError_t launch_lines_kernel(const LineDev& d, int P, int64_t blocks, hipStream_t s) {
  switch (P) {
    case 1: return launch_P<T, RED, SPEC, 256, 1>(d, blocks, s);
    case 2: return launch_P<T, RED, SPEC, 256, 2>(d, blocks, s);
    case 4: return launch_P<T, RED, SPEC, 256, 4>(d, blocks, s);
    case 8: return launch_P<T, RED, SPEC, 256, 8>(d, blocks, s);
    case 16: return launch_P<T, RED, SPEC, 256, 16>(d, blocks, s);
    case 32: return launch_P<T, RED, SPEC, 256, 32>(d, blocks, s);
    case 64: return launch_P<T, RED, SPEC, 256, 64>(d, blocks, s);
    case 128: return launch_P<T, RED, SPEC, 256, 128>(d, blocks, s);
    case 256: return launch_P<T, RED, SPEC, 256, 256>(d, blocks, s);
    case 512: return launch_P<T, RED, SPEC, 512, 512>(d, blocks, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace linek

}  // namespace helm
