// Batched strided DFT passes for gfx950.
//
// The forward eigen-transform of the periodic auxiliary problem is a DFT
// along a periodised axis with F[l, i] = e^{-2 pi i l i / n} (the eigenvector
// matrix of the circulant pencil, eq. (eigvectorsPer)), and the final
// transform is its inverse with the 1/n factor (eq. (step3IFFTz3coeff)).  The
// periodised axes are never the contiguous one, so each pass works on a tile
// [L][W] = (transform axis) x (W consecutive contiguous columns): global loads
// and stores are W*sizeof(complex) contiguous bytes per row, and the L-point
// transform runs as Stockham radix-2/4/8 stages through LDS.  The first stage
// reads global memory and the last stage writes it, so a pass touches HBM
// exactly once each way.  Long axes are split into two passes (four-step:
// n = n_a n_b, twiddle e^{-2 pi i a c/n} between the passes).
#include <algorithm>
#include <atomic>

#include "helm_internal.h"

namespace helm {

namespace {

constexpr int kFftThreads = 256;
#ifndef HELM_FFT_TILE_BYTES
#define HELM_FFT_TILE_BYTES 32768
#endif
#ifndef HELM_FFT_MAX_W
#define HELM_FFT_MAX_W 32
#endif
constexpr int kFftLdsBytes = HELM_FFT_TILE_BYTES;
constexpr int kFftMaxW = HELM_FFT_MAX_W;

template <typename C> struct RealOf;
template <> struct RealOf<double2> { using T = double; };
template <> struct RealOf<float2> { using T = float; };

template <typename C> __device__ inline C load_as(const void* base, int64_t idx, int kind) {
  if (kind == ST_C128) {
    const double2 v = reinterpret_cast<const double2*>(base)[idx];
    C r;
    r.x = (typename RealOf<C>::T)v.x;
    r.y = (typename RealOf<C>::T)v.y;
    return r;
  }
  const float2 v = reinterpret_cast<const float2*>(base)[idx];
  C r;
  r.x = (typename RealOf<C>::T)v.x;
  r.y = (typename RealOf<C>::T)v.y;
  return r;
}

template <typename C> __device__ inline void store_as(void* base, int64_t idx, int kind, C v, int acc) {
  if (kind == ST_C128) {
    double2* p = reinterpret_cast<double2*>(base) + idx;
    double2 w = make_double2((double)v.x, (double)v.y);
    if (acc) {
      const double2 o = *p;
      w.x += o.x;
      w.y += o.y;
    }
    *p = w;
  } else {
    float2* p = reinterpret_cast<float2*>(base) + idx;
    float2 w = make_float2((float)v.x, (float)v.y);
    if (acc) {
      const float2 o = *p;
      w.x += o.x;
      w.y += o.y;
    }
    *p = w;
  }
}

// multiply by (sign * i)
template <typename C> __device__ inline C mul_si(C a, int sign) {
  C r;
  if (sign > 0) { r.x = -a.y; r.y = a.x; }
  else { r.x = a.y; r.y = -a.x; }
  return r;
}

template <int R, typename C> __device__ inline void dft(C* v, int sign);

template <> __device__ inline void dft<2, double2>(double2* v, int) {
  const double2 a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}
template <> __device__ inline void dft<2, float2>(float2* v, int) {
  const float2 a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}

template <typename C> __device__ inline void dft4(C& x0, C& x1, C& x2, C& x3, int sign) {
  const C a = cadd(x0, x2), b = csub(x0, x2), c = cadd(x1, x3), d = mul_si(csub(x1, x3), sign);
  x0 = cadd(a, c);
  x1 = cadd(b, d);
  x2 = csub(a, c);
  x3 = csub(b, d);
}

template <> __device__ inline void dft<4, double2>(double2* v, int sign) { dft4(v[0], v[1], v[2], v[3], sign); }
template <> __device__ inline void dft<4, float2>(float2* v, int sign) { dft4(v[0], v[1], v[2], v[3], sign); }

template <typename C> __device__ inline void dft8(C* v, int sign) {
  using T = typename RealOf<C>::T;
  C e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
  C o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
  dft4(e0, e1, e2, e3, sign);
  dft4(o0, o1, o2, o3, sign);
  const T c = (T)0.70710678118654752440;
  // w^1 = c(1 + s i), w^2 = s i, w^3 = c(-1 + s i)
  C t1, t3;
  {
    const C si = mul_si(o1, sign);
    t1.x = c * (o1.x + si.x);
    t1.y = c * (o1.y + si.y);
  }
  const C t2 = mul_si(o2, sign);
  {
    const C si = mul_si(o3, sign);
    t3.x = c * (si.x - o3.x);
    t3.y = c * (si.y - o3.y);
  }
  v[0] = cadd(e0, o0);
  v[4] = csub(e0, o0);
  v[1] = cadd(e1, t1);
  v[5] = csub(e1, t1);
  v[2] = cadd(e2, t2);
  v[6] = csub(e2, t2);
  v[3] = cadd(e3, t3);
  v[7] = csub(e3, t3);
}
template <> __device__ inline void dft<8, double2>(double2* v, int sign) { dft8(v, sign); }
template <> __device__ inline void dft<8, float2>(float2* v, int sign) { dft8(v, sign); }

// 3-point DFT with w = e^{sign 2 pi i / 3} = -1/2 + sign i sqrt(3)/2:
// X0 = x0 + (x1 + x2), X1,2 = x0 - (x1 + x2)/2 +- sign i (sqrt(3)/2)(x1 - x2).
template <typename C> __device__ inline void dft3(C* v, int sign) {
  using T = typename RealOf<C>::T;
  const T h = (T)0.86602540378443864676;  // sqrt(3)/2
  const C t1 = cadd(v[1], v[2]), t2 = csub(v[1], v[2]);
  C m;
  m.x = v[0].x - (T)0.5 * t1.x;
  m.y = v[0].y - (T)0.5 * t1.y;
  C q = mul_si(t2, sign);
  q.x *= h;
  q.y *= h;
  v[0] = cadd(v[0], t1);
  v[1] = cadd(m, q);
  v[2] = csub(m, q);
}
template <> __device__ inline void dft<3, double2>(double2* v, int sign) { dft3(v, sign); }
template <> __device__ inline void dft<3, float2>(float2* v, int sign) { dft3(v, sign); }

struct PassDev {
  int sign, acc, in_kind, out_kind;
  const void* cmode;
  const int* skip;
  const void* cin;
  const void* cout;
  int64_t chirp_n, chirp_na, chirp_S;
  int64_t cq;  // col / chirp_S of the thread (0 in a one-pass convolution)
  int tw4_mode, conj_out;
  int64_t I, od, in_so, in_sj, out_so1, out_so2, out_sk, tw4_S;
  int64_t ntile;  // tiles along I
  int64_t i_first = 0;  // first column of a convolution pass
  double scale_c;
  const void* tw;
  const void* tw4;
  const double* scale;
};

// Compile-time Stockham plan of a power-of-two length L: one radix-2 or -4
// stage first when log2(L) is not a multiple of 3, then radix-8 stages.
// Lengths 9 * 2^k (the convolution pass of a chirp-z transform of length
// 9 * 2^j) take the power-of-two stages of 2^k followed by two radix-3
// stages.
constexpr int ilog2(int L) { return L <= 1 ? 0 : 1 + ilog2(L / 2); }
constexpr bool has9(int L) { return L % 9 == 0; }
constexpr int p2part(int L) { return has9(L) ? L / 9 : L; }
constexpr int nst2(int L2) { return ilog2(L2) / 3 + (ilog2(L2) % 3 ? 1 : 0); }
constexpr int nstages(int L) { return nst2(p2part(L)) + (has9(L) ? 2 : 0); }
constexpr int radix_of(int L, int s) {
  return s >= nst2(p2part(L)) ? 3
                              : ((ilog2(p2part(L)) % 3 && s == 0) ? (ilog2(p2part(L)) % 3 == 1 ? 2 : 4) : 8);
}
constexpr int pow2_floor(int x) { return x < 2 ? 1 : 2 * pow2_floor(x / 2); }
// Columns per tile: an LDS tile of L x W complex values, W <= kFftMaxW.
// 32 KB tiles keep several blocks resident per compute unit.  The longest
// passes (L = 512) take 128 KB tiles (16 complex128 columns: 256-byte row
// segments) with 1024 threads, one block per compute unit: against 64 KB
// tiles of 256 threads (128-byte segments, two blocks) the pass over a
// 512^3 x 16 volume takes 17% less time.
constexpr int tile_bytes(int L) { return L >= 512 ? 4 * kFftLdsBytes : kFftLdsBytes; }
constexpr int threads_of(int L) { return L >= 512 ? 4 * kFftThreads : kFftThreads; }
template <typename C> constexpr int tile_w(int L) {
  return pow2_floor((tile_bytes(L) / (L * (int)sizeof(C))) < kFftMaxW ? tile_bytes(L) / (L * (int)sizeof(C))
                                                                       : kFftMaxW);
}
// A second tile for the complex64 512-point pass, chosen per plan by the
// tuner: 64 KB (16 columns, 128-byte row segments) with the same 1024
// threads, so that two blocks share a compute unit and one block's loads
// overlap the other's LDS stages.  WO = 0 is the default tile.
//
// A third, narrow tile (WO = -1) for launches that would have fewer blocks than
// the device has compute units: 8 values per thread in blocks of 64 to 256
// threads, so a quarter to a sixteenth of the columns per block (row segments of
// at least 16 bytes).  The short segments cost bandwidth, which a launch of that
// size does not use: the 1024-point convolution of 513 x 200 x 4 complex64 took
// 24 us in 52 blocks of 16 columns and in 200 of 4, 14 us in 400 of 2.
constexpr int narrow_threads(int L) { return L >= 512 ? 256 : (L >= 256 ? 128 : 64); }
template <typename C> constexpr int narrow_w(int L) {
  return pow2_floor(std::max(narrow_threads(L) * 8 / L, 16 / (int)sizeof(C)));
}
//
// Single passes over 1024 to 4096 points: the 128 KB tile holds 2 to 8
// complex128 columns, a 64 KB tile (WO = -2, 512 threads, two blocks per compute
// unit) half of them; the plan's tuner times both against two passes.
constexpr int kHalf = -2;
// The narrow tile of 512 threads for the last columns of a convolution over 2048
// or 4096 points (launch_conv_L), which run alone: one column of 4096
// complex128 points in 19 us, with 256 threads 21.
constexpr int kTail = -3;
template <typename C> constexpr int tail_w(int L) { return std::max(512 * 8 / L, 16 / (int)sizeof(C)); }
template <int L, typename C, int WO> constexpr int tile_w_of() {
  return WO == kHalf   ? tile_w<C>(L) / 2
         : WO == kTail ? tail_w<C>(L)
                       : (WO < 0 ? narrow_w<C>(L) : (WO ? WO : tile_w<C>(L)));
}
template <int L, int WO> constexpr int threads_for() {
  return WO == kHalf || WO == kTail ? 512 : (WO < 0 ? narrow_threads(L) : threads_of(L));
}
template <int L, typename C, int WO> constexpr int min_waves_of() { return WO > 0 ? 8 : (WO == kHalf ? 4 : 1); }

// LDS position of element (row, w) of a tile.  Rows of less than 128 bytes
// (half the bank cycle) get one pad element per 8: the first stage writes every
// eighth row, which would otherwise meet in the same banks (8 W elements apart;
// padded 9 W).
template <int W, typename C> constexpr bool padded() { return W * (int)sizeof(C) < 128; }
template <int W, typename C> __device__ inline int lpos(int row, int w) {
  const int e = row * W + w;
  return padded<W, C>() ? e + (e >> 3) : e;
}
template <int L, int W, typename C> constexpr int lds_elems() { return padded<W, C>() ? L * W + (L * W >> 3) : L * W; }

// Blocks are dealt to the 8 XCDs in turn, each with its own L2.  Tiles of row
// segments shorter than a cache line are renumbered so that an XCD takes a
// contiguous range of them: neighbours then find the rest of their lines in
// its L2.  A bijection on [0, n) for any n.
template <int W, typename C> __device__ inline int64_t tile_of_block(int64_t b, int64_t n) {
  if constexpr (W * (int)sizeof(C) >= 128) return b;
  const int64_t q = n / 8, r = n % 8, x = b % 8, k = b / 8;
  return x < r ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

// One Stockham stage of radix R with Ns points already combined.  Thread
// tid of NT owns butterflies t = tid + q*NT, t -> (j = t / W,
// w = t % W); since W divides NT, w = tid % W for every q.  All reads of a
// stage precede the barrier and all writes follow it, so the stage works in
// place in LDS.  The first stage reads global memory, the last writes it
// (with the four-step twiddle, the per-mode scale and the optional
// accumulation).
// What a stage loads from memory besides the data (the roots, and in the last
// forward stage of a convolution the transformed kernel) is loaded before the
// LDS reads and the barrier, so that its latency passes during them; row
// addresses advance by uniform strides from one 64-bit product per butterfly.
template <int L, int W, int NT, int R, int Ns, bool FIRST, bool LAST, typename C, bool GIN = true, bool GOUT = true,
          bool REG = false>
__device__ inline void stage(const PassDev& p, C* sm, const void* in, void* out, int64_t o, int64_t i0,
                             int64_t oq, int64_t orr, int64_t a4, const C* vin, int tid) {
  constexpr bool LOADG = FIRST && GIN;    // this stage reads global memory
  constexpr bool STOREG = LAST && GOUT;   // this stage writes global memory
  constexpr bool KERN = LAST && !GOUT;    // end of a convolution's forward transform
  constexpr int LR = L / R;
  constexpr int NBF = LR * W;
  static_assert(NT % W == 0 && lds_elems<L, W, C>() * (int)sizeof(C) <= 160 * 1024, "tile does not fit the thread block or LDS");
  constexpr int NB = (NBF + NT - 1) / NT;
  constexpr int step = L / (Ns * R);
  const int w = tid % W;
  const int64_t col = i0 + w;
  const bool colok = col < p.I;
  const C* tw = reinterpret_cast<const C*>(p.tw);
  C v[NB][R], tv[NB][R], hv[KERN ? NB : 1][KERN ? R : 1];
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int t = tid + q * NT;
    if (NB * NT == NBF || t < NBF) {
      const int j = t / W, k = j % Ns;
      if constexpr (Ns > 1) {
#pragma unroll
        for (int r = 1; r < R; ++r) tv[q][r] = tw[r * k * step];
      }
      if constexpr (KERN) {
        const C* hk = reinterpret_cast<const C*>(p.cmode) + orr + p.od * ((j / Ns) * Ns * R + k);
#pragma unroll
        for (int r = 0; r < R; ++r) hv[q][r] = hk[p.od * (r * Ns)];
      }
    }
  }
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int t = tid + q * NT;
    if (NB * NT == NBF || t < NBF) {
      const int j = t / W;
      if constexpr (LOADG && REG) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[q][r] = vin[q * R + r];  // loaded by the caller
      } else if constexpr (LOADG) {
        const int64_t off = o * p.in_so + (int64_t)j * p.in_sj + col, rs = LR * p.in_sj;
        if (p.cin) {
          const int64_t xr = p.cq + p.chirp_na * j, xs = p.chirp_na * LR;
          const C* ci = reinterpret_cast<const C*>(p.cin) + xr;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            C x;
            x.x = 0;
            x.y = 0;
            if (colok && xr + r * xs < p.chirp_n) x = cmul(load_as<C>(in, off + r * rs, p.in_kind), ci[r * xs]);
            v[q][r] = x;
          }
        } else {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            C x;
            x.x = 0;
            x.y = 0;
            if (colok) x = load_as<C>(in, off + r * rs, p.in_kind);
            v[q][r] = x;
          }
        }
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) v[q][r] = sm[lpos<W, C>(j + r * LR, w)];
      }
    }
  }
  if constexpr (!LOADG) __syncthreads();
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int t = tid + q * NT;
    if (NB * NT == NBF || t < NBF) {
      const int j = t / W;
      const int k = j % Ns;
      if constexpr (Ns > 1) {
#pragma unroll
        for (int r = 1; r < R; ++r) v[q][r] = cmul(v[q][r], tv[q][r]);
      }
      dft<R, C>(v[q], p.sign);
      const int base = (j / Ns) * Ns * R + k;
      if constexpr (!STOREG) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if constexpr (KERN) {
            v[q][r] = cmul(v[q][r], hv[q][r]);
            v[q][r].y = -v[q][r].y;
          }
          sm[lpos<W, C>(base + r * Ns, w)] = v[q][r];
        }
      } else {
        if (colok) {
          const int64_t oi0 = oq * p.out_so1 + orr * p.out_so2 + (int64_t)base * p.out_sk + col, os = Ns * p.out_sk;
          // mode index of the per-mode factors: the chirp row map when folding
          // a chirp, else the pass's own output index
          const int64_t mi0 = p.cout ? p.cq + p.chirp_na * base : orr + p.od * base;
          const int64_t ms = (p.cout ? p.chirp_na : p.od) * Ns;
          // Accumulating over 1024 and more points, one block of 1024 threads
          // per compute unit: all old values are loaded before the first
          // store (a store may alias the next load, so loads between the
          // stores are waited for one by one; 2048^2 mixed: 470 -> 458 us a
          // solve).  Smaller tiles have other blocks to hide those waits, and
          // the registers would cost occupancy; in the streaming pass these
          // loads would wait for the prefetch (512^3 x 4: 4.5 -> 5.3 ms).
          constexpr bool EARLY = L > 512 && !REG;
          const bool early = EARLY && p.acc && p.out_kind == ST_C128;
          double2 old[EARLY ? R : 1];
          if (EARLY && early) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
              const bool ok = !p.cout || mi0 + r * ms < p.chirp_n;
              old[EARLY ? r : 0] = ok ? reinterpret_cast<const double2*>(out)[oi0 + r * os] : make_double2(0, 0);
            }
          }
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const int kk = base + r * Ns;  // output frequency of this pass
            const int64_t mi = mi0 + r * ms, oi = oi0 + r * os;
            if (p.cout && mi >= p.chirp_n) continue;  // rows past the transform length are not stored
            C y = v[q][r];
            if (p.conj_out) y.y = -y.y;
            if (p.tw4) {
              // kk < L and the multiplier < n / L, so the index stays below n
              const C* t4 = reinterpret_cast<const C*>(p.tw4);
              y = cmul(y, t4[kk * (p.tw4_mode ? orr : a4)]);
            }
            if (p.cmode) y = cmul(y, reinterpret_cast<const C*>(p.cmode)[mi]);
            if (p.cout) y = cmul(y, reinterpret_cast<const C*>(p.cout)[mi]);
            double s = p.scale_c;
            if (p.scale) s *= p.scale[mi];
            y.x = (typename RealOf<C>::T)(y.x * s);
            y.y = (typename RealOf<C>::T)(y.y * s);
            if (EARLY && early)
              reinterpret_cast<double2*>(out)[oi] =
                  make_double2((double)y.x + old[EARLY ? r : 0].x, (double)y.y + old[EARLY ? r : 0].y);
            else
              store_as<C>(out, oi, p.out_kind, y, p.acc);
          }
        }
      }
    }
  }
  if constexpr (!STOREG) __syncthreads();
}

template <int L, int W, int NT, int S, int Ns, typename C, bool GIN = true, bool GOUT = true, bool REG = false>
__device__ inline void stages(const PassDev& p, C* sm, const void* in, void* out, int64_t o, int64_t i0,
                              int64_t oq, int64_t orr, int64_t a4, const C* vin = nullptr,
                              int tid = (int)threadIdx.x) {
  if constexpr (S < nstages(L)) {
    constexpr int R = radix_of(L, S);
    stage<L, W, NT, R, Ns, S == 0, S == nstages(L) - 1, C, GIN, GOUT, REG>(p, sm, in, out, o, i0, oq, orr, a4, vin,
                                                                           tid);
    stages<L, W, NT, S + 1, Ns * R, C, GIN, GOUT, REG>(p, sm, in, out, o, i0, oq, orr, a4, vin, tid);
  }
}

// Quotient of a column by a positive 64-bit divisor: 32-bit where it fits (a
// 64-bit division is about a hundred instructions).
__device__ inline int64_t col_div(int64_t col, int64_t d) {
  if ((uint64_t)col >> 32 || (uint64_t)d >> 32) return col / d;
  return (uint32_t)col / (uint32_t)d;
}

// PLAIN: a single pass of a power-of-two axis, without chirp, four-step twiddle
// or per-mode complex factor (checked by the launcher and set here as
// constants, so that no stage carries their branches).
template <int L, typename C, int WO, bool PLAIN>
__global__ __launch_bounds__((threads_for<L, WO>()), (min_waves_of<L, C, WO>())) void fft_pass_kernel(PassDev p0,
                                                                                                     const void* in,
                                                                                                     void* out) {
  constexpr int W = tile_w_of<L, C, WO>(), NT = threads_for<L, WO>();
  __shared__ C sm[nstages(L) > 1 ? lds_elems<L, W, C>() : 1];
  if (p0.skip && *p0.skip) return;
  PassDev p = p0;
  const uint32_t blk = (uint32_t)tile_of_block<W, C>(blockIdx.x, gridDim.x), nt = (uint32_t)p.ntile;
  const uint32_t o = blk / nt;
  const int64_t i0 = (int64_t)(blk - o * nt) * W;
  const int64_t col = i0 + (int64_t)(threadIdx.x % W);
  int64_t oq = o, orr = 0, a4 = 0;
  if constexpr (PLAIN) {
    p.cin = p.cout = p.cmode = p.tw4 = nullptr;
    p.conj_out = 0;
    p.od = 1;
  } else {
    if (p.od > 1) {
      oq = o / (uint32_t)p.od;
      orr = o - oq * p.od;
    }
    if (p.tw4 && !p.tw4_mode) a4 = col_div(col, p.tw4_S);
    if (p.cin || p.cout) p.cq = col_div(col, p.chirp_S);
  }
  stages<L, W, NT, 0, 1, C>(p, sm, in, out, o, i0, oq, orr, a4);
}

// Streaming form of the 512-point pass (the plan's tile choice 2): one
// block per compute unit walks the tiles blk, blk + G, blk + 2G, ... and
// issues the loads of its next tile's first-stage inputs into registers
// right after the first stage of the current one, so each compute unit
// keeps HBM reads in flight through the remaining LDS stages and the
// stores.  (With one block per tile, a compute unit holding a single 128 KB
// tile leaves HBM idle for the length of its LDS stages.)  The global
// loads of a wave complete in issue order, so waiting for any load issued
// after the prefetch would wait for the prefetch too: the stage twiddles
// and the per-mode scale are therefore read from LDS copies made once per
// block, and the loads are unconditional (columns past the end read column
// 0 of the row, in bounds) and masked when the values are taken.  Inputs
// in the compute precision; no chirp factors, per-mode multiplier,
// conjugation or four-step twiddle, and od = 1 (single passes over the
// axis; checked by the launcher and set here as constants, so that the
// epilogue keeps only the scale).  The output kind and the accumulation
// are template arguments, so that the stores are straight-line code and the
// compiler's wait for the prefetched values at the top of the loop does not
// also wait for the previous tile's stores.  TIN is the input element
// (complex128 input of a complex64 pass: W = 16 columns, so that the
// prefetched complex128 values take the registers of 32 complex64 ones).
template <int L, typename C, typename TIN, int W, bool OUT128, bool ACC>
__global__ __launch_bounds__(threads_of(L), 1) void fft_stream_kernel(PassDev p0, const void* in, void* out,
                                                                      int64_t ntot) {
  using T = typename RealOf<C>::T;
  constexpr int NT = threads_of(L);
  constexpr int R0 = radix_of(L, 0);
  constexpr int LR = L / R0;
  constexpr int NB = LR * W / NT;
  static_assert(NB * NT == LR * W, "the first stage's butterflies fill the block");
  static_assert((lds_elems<L, W, C>() + L) * sizeof(C) + L * sizeof(double) <= 160 * 1024, "LDS");
  __shared__ C sm[lds_elems<L, W, C>()];
  __shared__ C twl[L];
  __shared__ double scl[L];
  if (p0.skip && *p0.skip) return;
  const int tid = threadIdx.x;
  const int w = tid % W;
  const int64_t G = gridDim.x;
  for (int e = tid; e < L; e += NT) {
    twl[e] = reinterpret_cast<const C*>(p0.tw)[e];
    scl[e] = p0.scale ? p0.scale[e] : 1.0;
  }
  PassDev p = p0;
  p.cin = p.cout = p.cmode = p.tw4 = nullptr;
  p.conj_out = 0;
  p.od = 1;
  p.out_kind = OUT128 ? ST_C128 : ST_C64;
  p.acc = ACC ? 1 : 0;
  p.tw = twl;
  p.scale = scl;
  TIN pre[NB * R0];
  // Row r LR + j of a tile: the tile's base (uniform) plus the thread's
  // 32-bit byte offset (j in_sj + w) sizeof(TIN) (the launcher checks that
  // LR in_sj sizeof(TIN) < 2^31), so that only the thread offsets take
  // vector registers besides the values.
  uint32_t toff[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q)
    toff[q] = (uint32_t)(((tid + q * NT) / W) * p.in_sj + w) * (uint32_t)sizeof(TIN);
  auto fetch = [&](int64_t tile) -> bool {
    const int64_t o = tile / p.ntile;
    const int64_t i0 = (tile - o * p.ntile) * W;
    const bool ok = i0 + w < p.I;
    const uint32_t msk = ok ? 0xffffffffu : 0u;
    const char* base = reinterpret_cast<const char*>(reinterpret_cast<const TIN*>(in) + o * p.in_so + i0);
#pragma unroll
    for (int r = 0; r < R0; ++r) {
      const char* br = base + (int64_t)r * LR * p.in_sj * (int64_t)sizeof(TIN);
#pragma unroll
      for (int q = 0; q < NB; ++q) pre[q * R0 + r] = *reinterpret_cast<const TIN*>(br + (toff[q] & msk));
    }
    return ok;
  };
  int64_t tile = blockIdx.x;
  bool ok = tile < ntot ? fetch(tile) : false;
  __syncthreads();  // the LDS copies of the tables
  for (; tile < ntot; tile += G) {
    C v[NB * R0];
#pragma unroll
    for (int k = 0; k < NB * R0; ++k) {
      v[k].x = ok ? (T)pre[k].x : (T)0;
      v[k].y = ok ? (T)pre[k].y : (T)0;
    }
    const int64_t o = tile / p.ntile;
    const int64_t i0 = (tile - o * p.ntile) * W;
    // The output row offsets (multiples of out_sk) and the LDS addresses
    // of the stages are the same for every tile; empty asm statements make
    // the stride and the thread index new to the compiler in each
    // iteration, so it recomputes those per tile instead of keeping all of
    // them in registers across the loop.
    int64_t osk = p0.out_sk;
    int tl = tid;
    asm volatile("" : "+s"(osk), "+v"(tl));
    p.out_sk = osk;
    // first stage from the registers into LDS, then the next tile's loads
    stage<L, W, NT, R0, 1, true, nstages(L) == 1, C, true, true, true>(p, sm, in, out, o, i0, o, 0, 0, v, tl);
    if (tile + G < ntot) ok = fetch(tile + G);
    stages<L, W, NT, 1, R0, C, true, true, true>(p, sm, in, out, o, i0, o, 0, 0, v, tl);
  }
}

// Chirp-z middle pass: forward DFT over the rows into LDS, multiplication by
// the transformed kernel and conjugation as its last stage writes them, a
// second forward DFT, and the conjugating epilogue: conj(DFT(conj(X))) is the
// unscaled inverse DFT.  ONE: L is the whole convolution length and the chirps
// are folded into the first load and the last store, so that the pass is the
// complete transform.
template <int L, typename C, int WO, bool ONE>
__global__ __launch_bounds__((threads_for<L, WO>())) void conv_pass_kernel(PassDev p0, const void* in, void* out) {
  constexpr int W = tile_w_of<L, C, WO>(), NT = threads_for<L, WO>();
  __shared__ C sm[lds_elems<L, W, C>()];
  if (p0.skip && *p0.skip) return;
  PassDev p = p0;
  const uint32_t blk = (uint32_t)tile_of_block<W, C>(blockIdx.x, gridDim.x), nt = (uint32_t)p.ntile;
  const uint32_t o = blk / nt;
  const int64_t i0 = p.i_first + (int64_t)(blk - o * nt) * W;
  int64_t oq = o, orr = 0;
  if constexpr (ONE) {
    p.od = 1;
    p.chirp_na = 1;
    p.tw4 = nullptr;
  } else {
    p.cin = p.cout = nullptr;
    if (p.od > 1) {
      oq = o / (uint32_t)p.od;
      orr = o - oq * p.od;
    }
  }
  stages<L, W, NT, 0, 1, C, true, false>(p, sm, in, out, o, i0, oq, orr, 0);
  p.cmode = nullptr;
  stages<L, W, NT, 0, 1, C, false, true>(p, sm, in, out, o, i0, oq, orr, 0);
}

// Compute units of the current device.  (Cached per device; threads that race
// on the first query store the same value.)
int compute_units() {
  static std::atomic<int> cu[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cu[dev].load(std::memory_order_relaxed);
  if (n <= 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cu[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Would a launch of the default tile leave compute units without a block, and
// does the narrow tile give more blocks?
template <int L, typename C> bool narrow_launch(const PassDev& p, int64_t O) {
  constexpr int W = tile_w<C>(L), WN = narrow_w<C>(L);
  return WN < W && p.I > WN && O * ((p.I + W - 1) / W) < compute_units();
}

// Columns [first, first + count) in tiles of WO.
template <int L, typename C, int WO>
hipError_t launch_conv_cols(const PassDev& p, int64_t O, int64_t first, int64_t count, const void* in, void* out,
                            hipStream_t s) {
  constexpr int W = tile_w_of<L, C, WO>();
  PassDev q = p;
  q.i_first = first;
  q.ntile = (count + W - 1) / W;
  const int64_t blocks = O * q.ntile;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 g((unsigned)blocks), b(threads_for<L, WO>());
  if (p.cin && p.cout && !p.tw4 && p.od == 1 && p.chirp_na == 1 && p.chirp_S >= p.I) {
    hipLaunchKernelGGL((conv_pass_kernel<L, C, WO, true>), g, b, 0, s, q, in, out);
  } else {
    if constexpr (L > 512) return hipErrorInvalidValue;  // middle passes are at most 512 rows long
    else {
      if (p.cin || p.cout) return hipErrorInvalidValue;
      hipLaunchKernelGGL((conv_pass_kernel<L, C, WO, false>), g, b, 0, s, q, in, out);
    }
  }
  return hipGetLastError();
}

// The 128 KB tiles run one per compute unit, in rounds.  Where the columns past
// the last full tile would open a round of their own (2^k + 1 columns: the
// paper's grids), they go to narrow tiles in a launch after the full ones, which
// take 11 to 19 us against a round of 20 to 30 (513^2 x 4 FP64 40 -> 35 us,
// 1025^2 x 4 mixed 110 -> 90, 257 x 2049 x 8 mixed 72 -> 57, 2049^2 FP64 127 -> 124).
template <int L, typename C> hipError_t launch_conv_L(const PassDev& p, int64_t O, const void* in, void* out, hipStream_t s) {
  if constexpr (L >= 64) {
    if (narrow_launch<L, C>(p, O)) return launch_conv_cols<L, C, -1>(p, O, 0, p.I, in, out, s);
  }
  if constexpr (L >= 512) {
    constexpr int WT = L == 2048 || L == 4096 ? kTail : -1;
    constexpr int W = tile_w<C>(L), WN = tile_w_of<L, C, WT>();
    const int64_t full = O * (p.I / W), rest = p.I % W, cu = compute_units();
    if (WN < W && rest > 0 && rest <= WN && full >= cu && (full + cu - 1) / cu < (full + O + cu - 1) / cu) {
      const hipError_t e = launch_conv_cols<L, C, 0>(p, O, 0, p.I - rest, in, out, s);
      if (e != hipSuccess) return e;
      return launch_conv_cols<L, C, WT>(p, O, p.I - rest, rest, in, out, s);
    }
  }
  return launch_conv_cols<L, C, 0>(p, O, 0, p.I, in, out, s);
}

template <typename C>
hipError_t launch_conv_typed(int L, const PassDev& p, int64_t O, const void* in, void* out, hipStream_t s) {
  switch (L) {
    case 9: return launch_conv_L<9, C>(p, O, in, out, s);
    case 18: return launch_conv_L<18, C>(p, O, in, out, s);
    case 36: return launch_conv_L<36, C>(p, O, in, out, s);
    case 72: return launch_conv_L<72, C>(p, O, in, out, s);
    case 2: return launch_conv_L<2, C>(p, O, in, out, s);
    case 4: return launch_conv_L<4, C>(p, O, in, out, s);
    case 8: return launch_conv_L<8, C>(p, O, in, out, s);
    case 16: return launch_conv_L<16, C>(p, O, in, out, s);
    case 32: return launch_conv_L<32, C>(p, O, in, out, s);
    case 64: return launch_conv_L<64, C>(p, O, in, out, s);
    case 128: return launch_conv_L<128, C>(p, O, in, out, s);
    case 256: return launch_conv_L<256, C>(p, O, in, out, s);
    case 512: return launch_conv_L<512, C>(p, O, in, out, s);
    // whole chirp-z convolutions in one pass (the plan's choice per axis)
    case 144: return launch_conv_L<144, C>(p, O, in, out, s);
    case 288: return launch_conv_L<288, C>(p, O, in, out, s);
    case 576: return launch_conv_L<576, C>(p, O, in, out, s);
    case 1152: return launch_conv_L<1152, C>(p, O, in, out, s);
    case 2304: return launch_conv_L<2304, C>(p, O, in, out, s);
    case 4608: return launch_conv_L<4608, C>(p, O, in, out, s);
    case 1024: return launch_conv_L<1024, C>(p, O, in, out, s);
    case 2048: return launch_conv_L<2048, C>(p, O, in, out, s);
    case 4096: return launch_conv_L<4096, C>(p, O, in, out, s);
    default: return hipErrorInvalidValue;
  }
}

template <int L, typename C, int WO = 0>
hipError_t launch_L(const PassDev& p, int64_t O, const void* in, void* out, hipStream_t s) {
  if constexpr (WO == 0 && L >= 64) {
    if (narrow_launch<L, C>(p, O)) return launch_L<L, C, -1>(p, O, in, out, s);
  }
  constexpr int W = tile_w_of<L, C, WO>();
  PassDev q = p;
  q.ntile = (p.I + W - 1) / W;
  const int64_t blocks = O * q.ntile;
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 g((unsigned)blocks), b(threads_for<L, WO>());
  if (!p.cin && !p.cout && !p.cmode && !p.tw4 && !p.conj_out && p.od == 1)
    hipLaunchKernelGGL((fft_pass_kernel<L, C, WO, true>), g, b, 0, s, q, in, out);
  else if constexpr (L <= 512)
    hipLaunchKernelGGL((fft_pass_kernel<L, C, WO, false>), g, b, 0, s, q, in, out);
  else
    return hipErrorInvalidValue;  // single passes of power-of-two axes only
  return hipGetLastError();
}

template <int L, typename C, typename TIN, int W>
hipError_t launch_stream_L(const PassDev& p, int64_t O, const void* in, void* out, hipStream_t s) {
  PassDev q = p;
  q.ntile = (p.I + W - 1) / W;
  const int64_t ntot = O * q.ntile;
  if (ntot <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>(ntot, compute_units());
  const dim3 g((unsigned)blocks), b(threads_of(L));
  const bool o128 = p.out_kind == ST_C128;
  if constexpr (sizeof(TIN) != sizeof(C)) {
    // complex128 input of a complex64 pass: complex64 output, no accumulation
    if (o128 || p.acc) return hipErrorInvalidValue;
    hipLaunchKernelGGL((fft_stream_kernel<L, C, TIN, W, false, false>), g, b, 0, s, q, in, out, ntot);
  } else {
    if (o128 && p.acc) hipLaunchKernelGGL((fft_stream_kernel<L, C, TIN, W, true, true>), g, b, 0, s, q, in, out, ntot);
    else if (o128) hipLaunchKernelGGL((fft_stream_kernel<L, C, TIN, W, true, false>), g, b, 0, s, q, in, out, ntot);
    else if (p.acc) hipLaunchKernelGGL((fft_stream_kernel<L, C, TIN, W, false, true>), g, b, 0, s, q, in, out, ntot);
    else hipLaunchKernelGGL((fft_stream_kernel<L, C, TIN, W, false, false>), g, b, 0, s, q, in, out, ntot);
  }
  return hipGetLastError();
}

// small_tile: 0 the default tile, 1 the 64 KB tile (complex64 at 512 points;
// 1024 to 4096 points), 2 the streaming pass (512 points; other passes and
// inputs that it does not take fall back to the default).
template <typename C>
hipError_t launch_typed(int L, const PassDev& p, int64_t O, const void* in, void* out, hipStream_t s,
                        int small_tile) {
  constexpr int kind = sizeof(C) == sizeof(float2) ? ST_C64 : ST_C128;
  if (L == 512 && small_tile == 2 && !p.cin && !p.cout && !p.cmode && !p.tw4 && !p.conj_out && p.od == 1) {
    constexpr int64_t LR = 512 / radix_of(512, 0);
    if (p.in_kind == kind && LR * p.in_sj * (int64_t)sizeof(C) < 0x7fffffffLL)
      return launch_stream_L<512, C, C, tile_w<C>(512)>(p, O, in, out, s);
    if constexpr (sizeof(C) == sizeof(float2)) {
      if (p.in_kind == ST_C128 && p.out_kind == ST_C64 && !p.acc && LR * p.in_sj * (int64_t)sizeof(double2) < 0x7fffffffLL)
        return launch_stream_L<512, C, double2, 16>(p, O, in, out, s);
    }
  }
  if constexpr (sizeof(C) == sizeof(float2)) {
    if (L == 512 && small_tile == 1) return launch_L<512, C, 16>(p, O, in, out, s);
  }
  if (small_tile == 1) {
    if (L == 1024) return launch_L<1024, C, kHalf>(p, O, in, out, s);
    if (L == 2048) return launch_L<2048, C, kHalf>(p, O, in, out, s);
    if (L == 4096) return launch_L<4096, C, kHalf>(p, O, in, out, s);
  }
  switch (L) {
    case 1024: return launch_L<1024, C>(p, O, in, out, s);
    case 2048: return launch_L<2048, C>(p, O, in, out, s);
    case 4096: return launch_L<4096, C>(p, O, in, out, s);
    case 2: return launch_L<2, C>(p, O, in, out, s);
    case 4: return launch_L<4, C>(p, O, in, out, s);
    case 8: return launch_L<8, C>(p, O, in, out, s);
    case 16: return launch_L<16, C>(p, O, in, out, s);
    case 32: return launch_L<32, C>(p, O, in, out, s);
    case 64: return launch_L<64, C>(p, O, in, out, s);
    case 128: return launch_L<128, C>(p, O, in, out, s);
    case 256: return launch_L<256, C>(p, O, in, out, s);
    case 512: return launch_L<512, C>(p, O, in, out, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int fft_tile_width(int L, bool fp32) { return fp32 ? tile_w<float2>(L) : tile_w<double2>(L); }

static PassDev make_pass_dev(const FftPass& f) {
  PassDev p;
  p.I = f.I;
  p.od = f.od;
  p.in_so = f.in_so;
  p.in_sj = f.in_sj;
  p.out_so1 = f.out_so1;
  p.out_so2 = f.out_so2;
  p.out_sk = f.out_sk;
  p.tw4_S = f.tw4_S;
  p.acc = f.accumulate;
  p.in_kind = f.in_kind;
  p.out_kind = f.out_kind;
  p.scale_c = f.scale_c;
  p.tw = f.tw;
  p.tw4 = f.tw4;
  p.scale = f.scale;
  p.sign = f.sign;
  p.cmode = f.cmode;
  p.skip = f.skip;
  p.cin = f.cin;
  p.cout = f.cout;
  p.chirp_n = f.chirp_n;
  p.chirp_na = f.chirp_na;
  p.chirp_S = f.chirp_S > 0 ? f.chirp_S : 1;
  p.tw4_mode = f.tw4_mode;
  p.conj_out = f.conj_out;
  p.cq = 0;
  p.ntile = 0;
  return p;
}

hipError_t launch_fft_pass(const FftPass& f, bool fp32, const void* in, void* out, hipStream_t s) {
  if (f.tw4 && f.tw4_mode == 0 && f.tw4_S <= 0) return hipErrorInvalidValue;
  const PassDev p = make_pass_dev(f);
  return fp32 ? launch_typed<float2>(f.L, p, f.O, in, out, s, f.small_tile)
              : launch_typed<double2>(f.L, p, f.O, in, out, s, f.small_tile);
}

hipError_t launch_conv_pass(const FftPass& f, bool fp32, const void* in, void* out, hipStream_t s) {
  if (!f.cmode) return hipErrorInvalidValue;
  const PassDev p = make_pass_dev(f);
  return fp32 ? launch_conv_typed<float2>(f.L, p, f.O, in, out, s)
              : launch_conv_typed<double2>(f.L, p, f.O, in, out, s);
}

}  // namespace helm
