// Fused line-transform kernels of the D-bar operator (included only by the per-N translation units).
//
// One application of A(S) = S + i F(q_k conj(h(S))) (paper Section 4, algorithm step 4, with Q -> q_k of Section 5.1)
// runs as six launches:
//   RowsInvScaled   F^{-1} S, first pass
//   ColsInvMoments  F^{-1} S, second pass, fused with the Taylor moments d_n = F(z^n s)(0)   (equation fourreeg4)
//   (moment reduction: d_n, c_n = (-i/2)^n d_n / n!, R(0) = (-i/2) F(conj(z) s)(0))
//   RowsInvRegular  R = (S - G)/xi with G of equation Gchoice, first pass of F^{-1} R
//   ColsInvTailFwd  second pass of F^{-1} R, h = F^{-1} R + sum c_n W_n (equation S0Taylor), u = q_k conj(h),
//                   first pass of F u  -- all in registers between the two column transforms
//   RowsFwdEpilogue second pass of F u and A(S) = S + i F(u)
//
// The same operator on s = F^{-1} S (the form the Krylov solver iterates on: F is unitary up to a constant, so GMRES
// takes the same steps, and the moments are sums over the x grid that need no transform) runs as three launches plus
// the moment reduction:
//   RowsFwdMoments      moments d_n = F(z^n s)(0), dt = F(conj(z) s)(0) of the input, first pass of F s
//   ColsFwdRegularInv   second pass of F s (= S), R = (S - G)/xi, first pass of F^{-1} R
//   RowsInvTailEpilogue second pass of F^{-1} R, h, and F^{-1} A(S) = s + i q_k conj(h)
//
// Every vector of that iteration is q_k times something (the right-hand side is -i q_k, the operator's second term
// i q_k conj(h)), so it lives where the potential does.  The three launches keep to the potential's index box
// (LineArgs::box): the row launches run its rows only and touch its columns only, the column launch reads and writes its
// rows of the transform array (rows outside are zero going in, and h is not needed there coming out, unless the caller
// wants h itself).  They are bound by memory, so they shorten with the box.  Measured at N = 1024, L = 5, a Gaussian
// potential (44% of the rows and columns), 8 FP32 entries per launch beside a second lane: RowsFwdMoments 69 -> 25 us,
// ColsFwdRegularInv 67 -> 40 us, RowsInvTailEpilogue 76 -> 27 us; the 16-k mixed solve 7.1 -> 3.8 ms.  At N = 512, 45
// entries, FP64, a sum of three Gaussians: 134 -> 47, 93 -> 73, 153 -> 85 us; 11.4 -> 7.7 ms.
#pragma once

#include "dbar_ctl.h"
#include "dbar_fft.h"
#include "dbar_launch.h"

namespace dbar {

// Smallest u beyond which e^{-u} sum_{k<=M} u^k/k! (times a safety factor 10) is below the rounding unit, so that
// P(n+1, u) = 1 exactly for every n <= M and omega_n = i / z^{n+1} (index M = 0..15).
static __constant__ float kTailOneF32[16] = {19.0f,  22.75f, 26.0f,  28.75f, 31.25f, 33.5f,  36.0f,  38.0f,
                                             40.25f, 42.25f, 44.25f, 46.25f, 48.0f,  50.0f,  51.75f, 53.75f};
static __constant__ double kTailOneF64[16] = {39.25, 43.75, 47.25, 50.5, 53.5, 56.25, 59.0, 61.5,
                                              64.0,  66.5,  68.75, 71.0, 73.25, 75.5, 77.5, 79.75};

// Exact binomial coefficients C(n, k), n, k <= kMaxM (Pascal's rule at compile time), and reciprocals 1/j of the
// integers (j < kNInv) for the tail recurrences, which would otherwise divide in every step.
struct BinomTable {
  double v[kMaxM + 1][kMaxM + 1];
};
constexpr BinomTable make_binom() {
  BinomTable t{};
  for (int n = 0; n <= kMaxM; ++n)
    for (int k = 0; k <= n; ++k) t.v[n][k] = (k == 0 || k == n) ? 1.0 : t.v[n - 1][k - 1] + t.v[n - 1][k];
  return t;
}
static __constant__ BinomTable kBinom = make_binom();

constexpr int kNInv = 256;
struct InvTable {
  double d[kNInv];
  float f[kNInv];
};
constexpr InvTable make_inv() {
  InvTable t{};
  for (int j = 1; j < kNInv; ++j) t.d[j] = 1.0 / j, t.f[j] = 1.0f / j;
  return t;
}
static __constant__ InvTable kInv = make_inv();
template <typename TT>
DBAR_D TT inv_int(int j) {
  if constexpr (sizeof(TT) == 8) return kInv.d[j];
  else return kInv.f[j];
}


// x_j = L(-pi + 2 pi j / N)
template <int N>
DBAR_D double xgrid(int j, double L) {
  return L * (-kPi + (2.0 * kPi / N) * j);
}
// the same in the arithmetic type TT (the FP32 operator evaluates its tail in FP32)
template <typename TT, int N>
DBAR_D TT xgrid_t(int j, double L) {
  if constexpr (sizeof(TT) == 8) return xgrid<N>(j, L);
  else return static_cast<float>(L) * (static_cast<float>(-kPi) + static_cast<float>(2.0 * kPi / N) * j);
}

// 1/r: FP64 division, or the hardware reciprocal (1 ulp) in FP32
template <typename TT>
DBAR_D TT recip(TT r) {
  if constexpr (sizeof(TT) == 8) return 1.0 / r;
  else return __builtin_amdgcn_rcpf(r);
}

// Coefficients c_k = prod_{j=1..k} (M+1)/(M+1+j) of F(u) = (M+1)! sum_k u^k/(M+1+k)! in powers of v = u/(M+1), and
// the number of terms after which the rest is below half a rounding unit of F for every v < 1 (FP32 or FP64), for
// the orders the tail is instantiated with (M = 11 and kMaxM).  Read from constant memory in a loop unrolled by four:
// fully unrolled, the compiler keeps every coefficient in a register; rolled, each step waits for its own read.
constexpr int kSerK32[2] = {25, 28}, kSerK64[2] = {40, 45};
struct SeriesTables {
  double d[2][45];
  float f[2][28];
};
constexpr SeriesTables make_series() {
  SeriesTables t{};
  for (int w = 0; w < 2; ++w) {
    const int M1 = (w == 0 ? 11 : kMaxM) + 1;
    double c = 1.0;
    for (int k = 0; k < 45; ++k) {
      if (k > 0) c = c * (double)M1 / (double)(M1 + k);
      t.d[w][k] = c;
      if (k < 28) t.f[w][k] = (float)c;
    }
  }
  return t;
}
static __constant__ SeriesTables kSeries = make_series();

// sum_{n=0}^{M} d_n omega_n(z),  omega_n = i P(n+1, u) / z^{n+1},  u = |z|^2/4  (c_n W_n = d_n omega_n).
// u <  M+1: omega_n = i E_n (conj(z)/4)^{n+1} with E_n = e^{-u} sum_k u^k/(n+1+k)!  (equation fourreg5a with the
//           factor e^{-u}); E_M by its series (a fixed-length polynomial), E_n = u E_{n+1} + e^{-u}/(n+1)! downwards
//           (positive terms only).
// u >= M+1: omega_n = i (1 - e^{-u} sum_{k<=n} u^k/k!) / z^{n+1}  (equation fourreg5); no cancellation there.
// TT is the arithmetic type: double in the FP64 operator, float in the FP32 one (whose data carry 24-bit mantissas).
// MM is the Taylor order the loops are unrolled for: the order M itself (M = 11, the paper's choice), or kMaxM for any
// M, which is exact too because d_n = 0 for M < n <= kMaxM.  d holds d_0..d_kMaxM in registers.
template <typename TT, int MM>
DBAR_D cx<TT> tail_sum(TT x, TT y, const cx<TT> (&d)[kMaxM + 1]) {
  const TT r2 = x * x + y * y;
  const TT u = TT(0.25) * r2;
  const TT one_from = sizeof(TT) == 8 ? TT(kTailOneF64[MM]) : TT(kTailOneF32[MM]);
  if (u >= one_from) {  // all P(n+1, u) = 1: i sum_n d_n / z^{n+1}
    const TT ir2 = recip(r2);
    const cx<TT> w{x * ir2, -y * ir2};
    cx<TT> acc = d[MM];
#pragma unroll
    for (int n = MM - 1; n >= 0; --n) acc = cfma(w, acc, d[n]);
    return mul_i(w * acc);
  }
  const TT eu = exp(-u);
  cx<TT> acc{TT(0), TT(0)};
  if (u < TT(MM + 1)) {
    // E_M = e^{-u} F(u) / (M+1)!, F(u) = sum_k c_k v^k with v = u/(M+1) < 1, c_k = prod_{j<=k} (M+1)/(M+1+j):
    // a fixed number of Horner steps (positive terms; the first omitted one is below half a rounding unit of F)
    static_assert(MM == 11 || MM == kMaxM, "series tables for M = 11 and kMaxM");
    constexpr int W = MM == 11 ? 0 : 1;
    constexpr int K = sizeof(TT) == 8 ? kSerK64[W] : kSerK32[W];
    const TT* c;
    if constexpr (sizeof(TT) == 8) c = kSeries.d[W];
    else c = kSeries.f[W];
    const TT v = u * TT(1.0 / (MM + 1));
    TT F = c[K - 1];
#pragma unroll 4
    for (int k = K - 2; k >= 0; --k) F = F * v + c[k];
    TT E = eu * F * TT(kInvFact[MM + 1]);
    const cx<TT> zeta{TT(0.25) * x, TT(-0.25) * y};
    acc = E * d[MM];
#pragma unroll
    for (int n = MM - 1; n >= 0; --n) {
      E = u * E + eu * TT(kInvFact[n + 1]);
      acc = cfma(zeta, acc, E * d[n]);
    }
    acc = zeta * acc;
  } else {
    TT P[MM + 1];
    TT t = eu, S = eu;
#pragma unroll
    for (int n = 0; n <= MM; ++n) {
      P[n] = TT(1) - S;
      t *= u * inv_int<TT>(n + 1);
      S += t;
    }
    const TT ir2 = recip(r2);
    const cx<TT> w{x * ir2, -y * ir2};  // 1/z
    acc = P[MM] * d[MM];
#pragma unroll
    for (int n = MM - 1; n >= 0; --n) acc = cfma(w, acc, P[n] * d[n]);
    acc = w * acc;
  }
  return mul_i(acc);
}

// The same sum from a table of what does not depend on the entry: e^{-u} and E_MM = P(MM+1, u)/u^{MM+1} at the point
// (tab = {e^{-u}, E_MM}, k_tail_table).  omega_n = i E_n (conj(z)/4)^{n+1} and E_n = u E_{n+1} + e^{-u}/(n+1)! hold for
// every u (positive terms only), so one recurrence serves up to where every P rounds to 1.  It leaves out the
// exponential, the series (40 dependent steps in FP64) and the division, which bounded the tail launch in FP64; the entry is
// one more 16-byte read per point, from L2 for all batch entries but the first.  Tail launch, before -> after: FP64 N = 128,
// 1 entry 12.7 -> 9.7 us, 1024 entries 182 -> 129; N = 256, 63 entries 36 -> 27; N = 512, 45 entries 77 -> 61; N = 1024,
// 8 entries 53 -> 43; FP32 N = 1024, 8 entries 24.8 -> 23.4.  Error against 64 bits as before (the table is FP64's own).
template <typename TT, int MM>
DBAR_D cx<TT> tail_tab(TT x, TT y, const cx<TT> (&d)[kMaxM + 1], cx<TT> tab) {
  const TT r2 = x * x + y * y;
  const TT u = TT(0.25) * r2;
  const TT one_from = sizeof(TT) == 8 ? TT(kTailOneF64[MM]) : TT(kTailOneF32[MM]);
  cx<TT> acc;
  if (u >= one_from) {  // all P(n+1, u) = 1: i sum_n d_n / z^{n+1}
    const TT ir2 = recip(r2);
    const cx<TT> w{x * ir2, -y * ir2};
    acc = d[MM];
#pragma unroll
    for (int n = MM - 1; n >= 0; --n) acc = cfma(w, acc, d[n]);
    acc = w * acc;
  } else {
    const cx<TT> zeta{TT(0.25) * x, TT(-0.25) * y};
    TT E = tab.im;
    acc = E * d[MM];
#pragma unroll
    for (int n = MM - 1; n >= 0; --n) {
      E = fmar(u, E, tab.re * TT(kInvFact[n + 1]));
      acc = cfma(zeta, acc, E * d[n]);
    }
    acc = zeta * acc;
  }
  return mul_i(acc);
}
// {e^{-u}, E_MM} at u in FP64 (E_MM by its series below u = MM + 1, from the closed form of P beyond)
template <int MM>
DBAR_D c64 tail_entry(double u) {
  const double eu = exp(-u);
  if (u < MM + 1) {
    constexpr int W = MM == 11 ? 0 : 1, K = kSerK64[W];
    const double v = u / (MM + 1);
    double F = kSeries.d[W][K - 1];
    for (int k = K - 2; k >= 0; --k) F = F * v + kSeries.d[W][k];
    return c64{eu, eu * F * kInvFact[MM + 1]};
  }
  double t = eu, S = eu, up = u;
  for (int k = 1; k <= MM; ++k) {
    t *= u * kInv.d[k];
    S += t;
    up *= u;
  }
  return c64{eu, (1.0 - S) / up};
}
// The table holds one quarter of the plane: |row - N/2|, |col - N/2| <= N/2 (the points of the grid mirror in both axes).
constexpr int tail_pitch(int N) { return N / 2 + 1; }
// entry i of the table (t32: rounded; either may be null), x = L 2 pi |j - N/2| / N
DBAR_D void tail_table_entry(int i, int N, double L, int M, c64* t64, c32* t32) {
  const int np = tail_pitch(N);
  const double h = L * (2.0 * kPi / N), x = h * (i % np), y = h * (i / np);
  const double u = 0.25 * (x * x + y * y);
  const c64 e = M == 11 ? tail_entry<11>(u) : tail_entry<kMaxM>(u);
  if (t64) t64[i] = e;
  if (t32) t32[i] = cvt<float>(e);
}
template <int N>
DBAR_D int tail_index(int row, int col) {
  const int r = row - N / 2, c = col - N / 2;
  return (r < 0 ? -r : r) * tail_pitch(N) + (c < 0 ? -c : c);
}

// ------------------------------------------------------------------------------------------------------------
// Block reduction of per-thread FP64 values into global partials dst[v * stride]
// ------------------------------------------------------------------------------------------------------------
template <int NT, int NV>
DBAR_D void block_reduce_store(const double (&vals)[NV], double* __restrict__ dst, size_t stride, double* scratch) {
  __syncthreads();  // scratch aliases the transform's LDS
  if constexpr (NT >= 64) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const double x = wsum(vals[v]);
      if (lane == 0) scratch[wave * NV + v] = x;
    }
    __syncthreads();
    for (int v = threadIdx.x; v < NV; v += NT) {
      double s = 0.0;
      for (int w = 0; w < NT / 64; ++w) s += scratch[w * NV + v];
      dst[v * stride] = s;
    }
  } else {
#pragma unroll
    for (int v = 0; v < NV; ++v) scratch[threadIdx.x * NV + v] = vals[v];
    __syncthreads();
    for (int v = threadIdx.x; v < NV; v += NT) {  // fewer threads than values in tiny blocks
      double s = 0.0;
      for (int t = 0; t < NT; ++t) s += scratch[t * NV + v];
      dst[v * stride] = s;
    }
  }
}

// ------------------------------------------------------------------------------------------------------------
// Tiling
// ------------------------------------------------------------------------------------------------------------
// Elements per thread of the line kernels (the radix of their passes), by stage, precision and grid size.  Sixteen
// need the fewest passes and exchanges; eight and four put two and four times as many waves on a line, each with a
// shorter serial chain (the tails above all) and fewer registers.  The choice depends on nothing but the stage, the
// precision and the grid size: an entry's result is the same in any batch.
constexpr int by_n(int N, int e32, int e64, int e128, int e256, int e512, int e1024, int e2048, int e4096) {
  return N <= 32 ? e32 : N <= 64 ? e64 : N <= 128 ? e128 : N <= 256 ? e256 : N <= 512 ? e512 : N <= 1024 ? e1024
         : N <= 2048 ? e2048 : e4096;
}
// Measured with the row tiles below, boxes of a sum of three Gaussians at L = 5 (one entry / a batch of 2^22 .. 2^25 points;
// launch times in us; 16 -> 8 -> 4 elements per thread; between figures within a few percent the whole solve decided):
//   tails, FP64: N = 256 17 -> 13 -> 11 / 41 -> 35 -> 37; N = 512 18 -> 14 -> 12 / 41 -> 37 -> 38;
//     N = 1024 22 -> 18 -> 16 / 68 -> 64 -> 69; N = 2048 59 -> 55 -> 68 / 158 -> 175 -> 240;
//     N = 4096 174 -> 221 -> 235 / 318 -> 416 -> 443
//   tails, FP32: N = 256 14 -> 11 -> 9 / 20 -> 21 -> 21; N = 512 15 -> 11 -> 10 / 21 -> 21 -> 21;
//     N = 1024 17 -> 14 -> 14 / 35 -> 35 -> 39; N = 2048 24 -> 26 -> 31 / 55 -> 61 -> 82;
//     N = 4096 74 -> 89 -> 131 / 138 -> 177 -> 257
//   moments, FP64: N = 256 14 -> 13 -> 12 / 36 -> 37 -> 40; N = 512 16 -> 15 -> 15 / 38 -> 38 -> 41;
//     N = 1024 18 -> 18 -> 18 / 65 -> 68 -> 76; N = 2048 39 -> 40 -> 47 / 118 -> 122 -> 150;
//     N = 4096 125 -> 169 -> 196 / 227 -> 316 -> 366
//   moments, FP32: N = 256 16 -> 12 -> 12 / 24 -> 19 -> 22; N = 512 17 -> 14 -> 13 / 24 -> 19 -> 22;
//     N = 1024 18 -> 15 -> 15 / 40 -> 33 -> 41; N = 2048 26 -> 22 -> 28 / 66 -> 58 -> 68;
//     N = 4096 82 -> 76 -> 123 / 160 -> 136 -> 219
//   division, FP64: N = 256 15 -> 12 -> 11 / 53 -> 48 -> 50; N = 512 16 -> 13 -> 13 / 47 -> 41 -> 53;
//     N = 1024 19 -> 19 -> 19 / 75 -> 75 -> 96; N = 2048 46 -> 47 -> 64 / 149 -> 152 -> 232;
//     N = 4096 187 -> 193 -> 340 / 369 -> 377 -> 682
//   division, FP32: N = 256 14 -> 11 -> 10 / 21 -> 21 -> 22; N = 512 14 -> 11 -> 12 / 21 -> 21 -> 25;
//     N = 1024 18 -> 17 -> 14 / 37 -> 46 -> 44; N = 2048 24 -> 30 -> 43 / 67 -> 81 -> 124;
//     N = 4096 73 -> 111 -> 152 / 135 -> 212 -> 290
// and of the stages on S itself (whole grids):
//   ColsInvMoments, FP64: N = 64 21 -> 14 -> 11 / 75 -> 41 -> 48; N = 256 12 -> 10 -> 10 / 36 -> 30 -> 36;
//     N = 1024 16 -> 15 -> 16 / 54 -> 52 -> 87; N = 2048 37 -> 37 -> 52 / 152 -> 159 -> 225
//   ColsInvTailFwd, FP64: N = 64 17 -> 11 -> 9 / 64 -> 49 -> 46; N = 256 19 -> 13 -> 11 / 71 -> 49 -> 49;
//     N = 512 23 -> 16 -> 14 / 74 -> 51 -> 59; N = 1024 29 -> 25 -> 23 / 126 -> 112 -> 136;
//     N = 2048 99 -> 93 -> 124 / 340 -> 366 -> 470
//   ColsInvTailFwd, FP32: N = 256 16 -> 12 -> 10 / 32 -> 30 -> 29; N = 512 20 -> 14 -> 14 / 35 -> 32 -> 42;
//     N = 1024 25 -> 21 -> 17 / 66 -> 74 -> 86; N = 2048 44 -> 45 -> 64 / 156 -> 161 -> 233
//   RowsInvRegular, FP64: N = 64 12 -> 9 -> 8 / 38 -> 32 -> 30; N = 512 13 -> 10 -> 9 / 34 -> 30 -> 30;
//     N = 1024 19 -> 17 -> 16 / 60 -> 53 -> 57; FP32: N = 512 11 -> 9 -> 8 / 20 -> 17 -> 25
//   RowsFwdEpilogue, FP64: N = 64 11 -> 10 -> 9 / 145 -> 141 -> 139; N = 512 16 -> 14 -> 14 / 137 -> 135 -> 135;
//     N = 2048 152 -> 141 -> 149 / 565 -> 542 -> 565
//   ColsFwdPlain, FP64: N = 512 9 -> 8 -> 9; N = 1024 13 -> 13 -> 14; N = 2048 32 -> 34 -> 39;
//     N = 4096 252 -> 235 -> 428
template <typename T, int N>
struct Ept {
  static constexpr bool D = sizeof(T) == 8;
  static constexpr int FWD_MOMENTS = D ? by_n(N, 4, 16, 8, 4, 8, 8, 16, 16) : by_n(N, 4, 4, 4, 4, 8, 8, 8, 16);
  static constexpr int TAIL_ROWS = D ? by_n(N, 4, 4, 4, 4, 4, 4, 16, 16) : by_n(N, 4, 4, 4, 4, 4, 16, 16, 16);
  static constexpr int REG_COLS = D ? by_n(N, 4, 8, 8, 8, 8, 8, 16, 16) : by_n(N, 4, 4, 4, 4, 8, 16, 16, 16);
  // the stages of the operator on S itself (one application, N = 64: 70 -> 38 us; N = 1024: 99 -> 87 us).  FP32 at N = 512
  // and 1024 takes eight for its batches: 64 mixed solves on S at N = 512 18.2 -> 16.8 -> 18.5 ms, 32 at N = 1024
  // 37.3 -> 36.0 -> 38.0 ms, one application at N = 1024 94 -> 75 -> 70 us.
  static constexpr int MOMENT_COLS = by_n(N, 4, 4, 4, 8, 8, 8, 16, 16);
  static constexpr int TAIL_COLS = D ? by_n(N, 4, 4, 4, 4, 4, 4, 16, 16) : by_n(N, 4, 4, 4, 4, 8, 8, 16, 16);
  // the row stages and the column stages with light work per element
  static constexpr int ROWS = D ? by_n(N, 4, 4, 4, 4, 4, 8, 16, 16) : by_n(N, 4, 4, 4, 4, 8, 8, 16, 16);
  static constexpr int COLS = by_n(N, 4, 4, 4, 8, 8, 8, 16, 16);
};

template <typename T, int N>
struct Tiling {
  using G = LineGeom<N, 16>;
  static constexpr int cmin(int a, int b) { return a < b ? a : b; }
  static constexpr int cmax(int a, int b) { return a > b ? a : b; }
  static constexpr int kLdsBudget = 150 * 1024;
  static constexpr int fit(int lines) {
    while (lines > 1 && lines * G::LDS_LINE * (int)sizeof(cx<T>) > kLdsBudget) lines /= 2;
    return lines;
  }
  // Lines of a row tile: enough blocks to spread one entry of a small grid over the chip, two lines in FP32 at N = 1024,
  // where each leaves half of a line of the tiled array
  static constexpr int ROWS = cmin(N, N <= 64 ? 16 : N <= 256 ? 4 : N <= 512 ? 2 : N <= 1024 && sizeof(T) == 4 ? 2 : 1);
  // (FP32 at N = 4096: the LDS holds four full-height lines, but a four-line tile needs more than the 128 VGPRs of
  // four waves per SIMD and spills 72 bytes per lane; two lines fit without a spill and run faster)
  static constexpr int COLS = sizeof(T) == 4 && N >= 4096 ? 2
                                                          : fit(cmin(N, cmax(64 / (int)sizeof(cx<T>), cmax(1, 64 / G::TPL))));
  // Column-tile variants for the tuner: 0 = COLS (the default), then the wider tiles COLS << 1, COLS << 2 while a block
  // of sixteen elements per thread has at most 1024 threads and the tile's lines fit the LDS budget, then the narrower
  // tile COLS / 2 (more blocks per CU where one full-height tile fills most of the LDS, as at N = 4096).
  static constexpr bool wide_ok(int c) {
    return c <= N && c * G::TPL <= 1024 && c * G::LDS_LINE * (int)sizeof(cx<T>) <= kLdsBudget;
  }
  static constexpr int NWIDE = wide_ok(COLS << 1) ? (wide_ok(COLS << 2) ? 2 : 1) : 0;
  static constexpr bool NARROW = COLS >= 2;
  static constexpr int variants() { return 1 + NWIDE + (NARROW ? 1 : 0); }
  template <int V>
  static constexpr int cols_v() { return V == 0 ? COLS : V <= NWIDE ? (COLS << V) : COLS / 2; }
  template <int V>
  static constexpr bool cols_valid() { return V < variants(); }
  // the columns a stage of E elements per thread takes of a variant: at most 1024 threads, and with moments at most
  // 512 / N on small grids (more blocks for the one entry an application has there, and the reduction's scratch)
  template <int E, int V, bool MOMENTS>
  static constexpr int cols_of() {
    return cmin(cmin(cols_v<V>(), MOMENTS ? cmin(16, cmax(4, 512 / N)) : N), 1024 / (N / cmin(N, E)));
  }
  // Tile width of the FP32 transform array (t_index): the default column tile, but at least 8 columns, so that the
  // row launches move 64-byte pieces.  At N = 4096 the column tile is 2 columns (4 at most); 2- or 4-column pieces
  // cost the row launches more (they leave partial lines) than the narrow column tiles gain from whole pieces.
  static constexpr int LAYOUT_W = COLS < 8 && N >= 8 ? 8 : COLS;
};

// Index of element (row, col) of the x-space operator's transform array (the output of its first launch, rewritten in
// place by the column launch, read by the last).  FP32: column-tile-major with tiles of Tiling::LAYOUT_W columns, each
// tile one contiguous N x LAYOUT_W block, so that the column launch reads and writes whole or partial lines of it and
// the row launches whole LAYOUT_W-element pieces; the width is a compile-time constant, so the per-thread addresses
// keep constant strides.  FP64: row-major (the tiled FP64 array measured slower).
template <typename T, int N>
DBAR_D size_t t_index(int row, int col) {
  if constexpr (sizeof(T) == 8) {
    return (size_t)row * N + col;
  } else {
    constexpr int TW = Tiling<T, N>::LAYOUT_W;
    return ((size_t)(col / TW) * N + row) * TW + (col % TW);
  }
}

// LDS of one line-kernel block: the line data, or the scratch of its reductions, whichever is larger
template <typename T, class G, int LINES, bool COLS, bool MOMENTS>
struct LdsSize {
  static constexpr int TPL = G::TPL;
  static constexpr int NT = LINES * TPL;
  static constexpr int kData = LINES * G::LDS_LINE * (int)sizeof(cx<T>);
  static constexpr int LN = LINES;
  static constexpr int kScratchReduce = (NT >= 64 ? NT / 64 : NT) * 2 * kNMom * (int)sizeof(double);
  // the moment reduction's groups (MomentsBase::finish_kk): runs of min(TPL, 64) lanes of a row; on a column tile
  // (wave, column) pairs when the block has whole waves and fewer than 64 columns, else single threads
  static constexpr int NG = COLS ? ((NT >= 64 && LN < 64) ? (NT / 64) * LN : NT) : NT / (TPL < 64 ? TPL : 64);
  static constexpr int kScratchMoments = !MOMENTS ? 0 : (NG * 2 * (kMaxM + 1) + LN * 2 * kNMom + LN * 2 * (kMaxM + 1)) * 8;
  static constexpr int kScratch = kScratchReduce > kScratchMoments ? kScratchReduce : kScratchMoments;
  static constexpr int kElems = ((kData > kScratch ? kData : kScratch) + (int)sizeof(cx<T>) - 1) / (int)sizeof(cx<T>);
};

// ------------------------------------------------------------------------------------------------------------
// Reads and writes on an index box: buffer accesses whose offset is moved out of the buffer outside the box, where the
// hardware returns zero or drops the store without memory traffic, so that the box costs no branch around each access
// ------------------------------------------------------------------------------------------------------------
using Rsrc = __amdgpu_buffer_rsrc_t;
constexpr uint32_t kOutside = 0x80000000u;  // beyond every array here (N <= 4096: at most 2^28 bytes per entry)

// the N x N array of one entry at p (the same for every lane of the wave)
template <typename T, int N>
DBAR_D Rsrc entry_rsrc(const cx<T>* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<cx<T>*>(p), 0, N * N * (int)sizeof(cx<T>), 0x00020000);
}
// element idx, or zero / nothing when !in
template <typename T>
DBAR_D cx<T> box_load(Rsrc r, uint32_t idx, bool in) {
  const uint32_t off = in ? idx * (uint32_t)sizeof(cx<T>) : kOutside;
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(cx<T>, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
  else return __builtin_bit_cast(cx<T>, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
template <typename T>
DBAR_D void box_store(Rsrc r, uint32_t idx, bool in, cx<T> v) {
  using V2 = unsigned __attribute__((ext_vector_type(2)));
  using V4 = unsigned __attribute__((ext_vector_type(4)));
  const uint32_t off = in ? idx * (uint32_t)sizeof(cx<T>) : kOutside;
  if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V2, v), r, off, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(V4, v), r, off, 0, 0);
}

// an entry's box (uniform over the block); always the whole grid below kBoxMinN
template <int N>
struct Box {
  int r0, r1, c0, c1;
  DBAR_D bool row(int i) const { return N < kBoxMinN || (i >= r0 && i < r1); }
  DBAR_D bool col(int j) const { return N < kBoxMinN || (j >= c0 && j < c1); }
};
template <int N>
DBAR_D Box<N> entry_box(const LineArgs& a, int b) {
  if (N < kBoxMinN || !a.box) return Box<N>{0, N, 0, N};
  const int* x = a.box + (size_t)b * a.box_bs;
  return Box<N>{x[0], x[1], x[2], x[3]};
}

// ------------------------------------------------------------------------------------------------------------
// Operations
// ------------------------------------------------------------------------------------------------------------
struct NoAcc {};

template <typename T, int N, int E>
struct OpBase {
  using G = LineGeom<N, E>;
  static constexpr bool ROLLED = false;  // heavy per-element epilogue: process through LDS in a rolled loop
  LineArgs a;
  // the blocks of one tile for every entry of the batch are dispatched together, on one XCD (k_lines): for stages
  // that read an array all entries share (the potential), whose rows then stay in that XCD's L2 while the entries pass
  static constexpr bool TILE_MAJOR = false;
  static constexpr bool OWN_COEF = false;
  DBAR_D bool active(int b) const { return a.act == nullptr || a.act[b] != 0; }
  DBAR_D const cx<T>* inp(int b) const { return static_cast<const cx<T>*>(a.in) + (size_t)b * a.in_bs; }
  DBAR_D cx<T>* outp(int b) const { return static_cast<cx<T>*>(a.out) + (size_t)b * a.out_bs; }
  template <class Acc> DBAR_D void mid(int, int, int, cx<T>&) const {}
  // finish (and dots): the tile's partials go to slot `slot` of ntiles
  template <int NT, class Acc> DBAR_D void finish(Acc&, int, int, int, int, double*) const {}
  // after the stores: dots over the values the stores left in the thread's registers (ops that define DOTS)
  static constexpr bool DOTS = false;
  // the op works on its loaded values before the first transform (loaded(acc, b, line, jt, v, tile, ntiles, scratch)
  // may change them; it must be called by all threads of the block)
  static constexpr bool LOADACC = false;
  // ROLLED stores: > 1: the op's store_all stores the thread's elements GROUP at a time, else store one at a time
  static constexpr int GROUP = 1;
  // the op leaves moment partials (its block reduction needs their scratch)
  static constexpr bool MOMENTS = false;
  // the op works on the entry's box (row launches cover its rows only); its load and loaded take the Pre
  static constexpr bool BOXED = false;
  // per-block data read once at kernel start, before any store (ops that need it define PRE and a Pre type)
  static constexpr bool PRE = false;
  struct Pre {};
  DBAR_D void prologue(int, Pre&) const {}
};

// out = IFFT_rows(phase * ci * in)
template <typename T, int N>
struct OpRowsInvScaled : OpBase<T, N, Ept<T, N>::ROWS> {
  static constexpr int DIR1 = +1;
  static constexpr bool TWO = false;
  using Acc = NoAcc;
  DBAR_D cx<T> load(int b, int row, int pos) const {
    const T f = static_cast<T>(((row + pos) & 1) ? -this->a.ci : this->a.ci);
    return f * this->inp(b)[(size_t)row * N + pos];
  }
  DBAR_D void store(Acc&, int b, int row, int pos, cx<T> v) const { this->outp(b)[(size_t)row * N + pos] = v; }
};

// Moments sum z^n s (n <= M) and sum conj(z) s of x-space values s, reduced in FP64.  Along a line one coordinate
// is fixed (x on a column, y on a row); each thread accumulates mu_k = sum t^k s over its elements (t the varying
// coordinate: real weights, k <= M) and the line's share of d_n = sum_k C(n,k) (fixed part)^(n-k) (t part)^k is
// formed once at the end: on a column d_n = sum_k C(n,k) x^{n-k} i^k mu_k, conj moment x mu_0 - i mu_1; on a row
// d_n = sum_k C(n,k) (iy)^{n-k} mu_k, conj moment mu_1 - iy mu_0 (the binomial terms exceed |z|^n by at most
// 2^{n/2}, i.e. < 50x at n = 11: a few ulps of FP64).
template <typename T, int N, bool ALONG_X, int E>
struct MomentsBase : OpBase<T, N, E> {
  using G = LineGeom<N, E>;
  static constexpr bool MOMENTS = true;
  static constexpr int NV = 2 * kNMom;
  static constexpr int NMU = 2 * (kMaxM + 1);  // mu_0 .. mu_kMaxM (re, im)
  // Moments are accumulated over a thread's elements (4 to 16) and its group's lanes in the transform's precision (the FP32
  // operator's s carries FP32 rounding anyway, and the regularisation is exact for any G coefficients); the sums over
  // groups and tiles and the binomial combination run in FP64.
  struct Acc {
    T v[NMU];  // mu_k = sum t^k s over this thread's elements
  };
  // the fixed coordinate of line `line`
  DBAR_D double fixed(int line) const { return xgrid<N>(line, this->a.L); }
  // s at position pos of line `line` into this thread's mu_k
  DBAR_D void add(Acc& acc, int b, int line, int pos, cx<T> v) const {
    cx<T> s = v;
    // shifted regularisation: Taylor coefficients at xi = a are moments of s e^{-i a.x} = s e_k (the varying
    // coordinate's factor here, the fixed one's in combine_one)
    if (this->a.shv) {
      const size_t o = (size_t)b * this->a.e_bs + pos;
      if constexpr (sizeof(T) == 8) s = s * (ALONG_X ? this->a.ex[o] : this->a.ey[o]);
      else s = s * (ALONG_X ? this->a.ex32[o] : this->a.ey32[o]);
    }
    (void)line;
    // mu_0..mu_KK with KK fixed at compile time: the order M = 11 itself, else kMaxM (the extra mu_k are unused);
    // mu_1 is always needed (conj moment)
    if (this->a.M == 11) accumulate<11>(acc, xgrid_t<T, N>(pos, this->a.L), s);
    else accumulate<kMaxM>(acc, xgrid_t<T, N>(pos, this->a.L), s);
  }
  template <int KK>
  DBAR_D static void accumulate(Acc& acc, T t, cx<T> s) {
    T tp = T(1);
#pragma unroll
    for (int k = 0; k <= KK; ++k) {
      acc.v[2 * k] += tp * s.re;
      acc.v[2 * k + 1] += tp * s.im;
      tp *= t;
    }
  }
  // all of the thread's loaded values v[s] (position jt + s TPL) into its mu_k, the order's branch taken once
  DBAR_D void add_loaded(Acc& acc, int b, int line, int jt, const cx<T>* v) const {
    if (this->a.M == 11) add_all<11>(acc, b, jt, v);
    else add_all<kMaxM>(acc, b, jt, v);
    (void)line;
  }
  template <int KK>
  DBAR_D void add_all(Acc& acc, int b, int jt, const cx<T>* v) const {
#pragma unroll
    for (int s = 0; s < G::RMAX; ++s) {
      const int pos = jt + s * G::TPL;
      cx<T> sv = v[s];
      if (this->a.shv) {
        const size_t o = (size_t)b * this->a.e_bs + pos;
        if constexpr (sizeof(T) == 8) sv = sv * (ALONG_X ? this->a.ex[o] : this->a.ey[o]);
        else sv = sv * (ALONG_X ? this->a.ex32[o] : this->a.ey32[o]);
      }
      accumulate<KK>(acc, xgrid_t<T, N>(pos, this->a.L), sv);
    }
  }
  // Moment q of one line from its mu_k (q <= M; 0 for M < q <= kMaxM; q = kMaxM+1: the conj moment), c its fixed
  // coordinate; with the shifted regularisation times the line's factor of e_k.  mu is (re, im) interleaved.
  DBAR_D c64 combine_one(const double* mu, double c, int q, int b, int line) const {
    double re = 0.0, im = 0.0;
    if (q == kMaxM + 1) {
      if constexpr (ALONG_X) {  // mu_1 - i y mu_0
        re = mu[2] + c * mu[1];
        im = mu[3] - c * mu[0];
      } else {  // x mu_0 - i mu_1
        re = c * mu[0] + mu[3];
        im = c * mu[1] - mu[2];
      }
    } else if (q <= this->a.M) {
      double cpow = 1.0;  // c^{q-k} for k = q, q-1, ..., 0
      for (int k = q; k >= 0; --k) {
        const double w = kBinom.v[q][k] * cpow;
        const double mr = mu[2 * k], mi = mu[2 * k + 1];
        switch ((ALONG_X ? q - k : k) & 3) {  // times i^k (column) or i^{q-k} (row)
          case 0: re += w * mr; im += w * mi; break;
          case 1: re -= w * mi; im += w * mr; break;
          case 2: re -= w * mr; im -= w * mi; break;
          default: re += w * mi; im -= w * mr; break;
        }
        cpow *= c;
      }
    }
    c64 d{re, im};
    if (this->a.shv) d = (ALONG_X ? this->a.ey : this->a.ex)[(size_t)b * this->a.e_bs + line] * d;
    return d;
  }

  template <int NT>
  DBAR_D void finish(Acc& acc, int b, int tile, int slot, int ntiles, double* scratch) const {
    if (this->a.M == 11) finish_kk<NT, 11>(acc, b, tile, slot, ntiles, scratch);
    else finish_kk<NT, kMaxM>(acc, b, tile, slot, ntiles, scratch);
  }
  // Block reduction: 1) each line's mu_k summed over its threads within a wave by shuffles (a column tile
  // interleaves its lines, so a column's lanes differ by multiples of LN; a row's lanes are contiguous), parked in
  // LDS per reduction group; 2) summed over the line's groups (one thread per line and value); 3) combined into the
  // moments (one thread per line and moment); 4) the tile's partials: sum over its lines.
  template <int NT, int KK>
  DBAR_D void finish_kk(Acc& acc, int b, int tile, int slot, int ntiles, double* scratch) const {
    constexpr int NU = 2 * (KK + 1);  // mu values in use
    double* dst = this->a.part + (size_t)b * NV * ntiles + slot;
    constexpr int TPL = G::TPL;
    constexpr int LN = NT / TPL;  // lines per tile
    // reduction groups: runs of GS consecutive lanes on a row tile; (wave, column) pairs on a column tile of fewer
    // than 64 columns (SHFL), else single threads
    constexpr int GS = ALONG_X ? (TPL < 64 ? TPL : 64) : 1;
    constexpr bool SHFL = !ALONG_X && NT >= 64 && LN < 64;
    constexpr int NG = ALONG_X ? NT / GS : SHFL ? (NT / 64) * LN : NT;
    static_assert(NG == LdsSize<T, G, LN, !ALONG_X, true>::NG, "LDS scratch sized for another reduction layout");
    __syncthreads();  // scratch aliases the transform's LDS
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double* sc = scratch;                 // [NG][NMU]
    double* colv = scratch + NG * NMU;    // [LN][NV]
    double* mus = colv + LN * NV;         // [LN][NMU]
    if constexpr (ALONG_X || SHFL) {
      // over the lanes of a group: halved as far as NU splits evenly (24 or 32 values over 64 lanes: 30 exchanges per
      // lane instead of 6 NU)
      constexpr int OFF = ALONG_X ? GS / 2 : 32, LAST = ALONG_X ? 1 : LN;
      const int base = reduce_lanes<NU, OFF, LAST>(acc.v, lane);
      const int g = ALONG_X ? threadIdx.x / GS : wave * LN + lane % LN;
      if ((lane & reduce_copies<NU, OFF, LAST>()) == 0) {
#pragma unroll
        for (int i = 0; i < reduce_left<NU, OFF, LAST>(); ++i) sc[g * NMU + base + i] = static_cast<double>(acc.v[i]);
      }
    } else {  // thread t serves column t % LN
#pragma unroll
      for (int q = 0; q < NU; ++q) sc[threadIdx.x * NMU + q] = static_cast<double>(acc.v[q]);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < LN * NU; t += NT) {
      const int c = t / NU, q = t % NU;
      double v = 0.0;
      if constexpr (ALONG_X) {
        constexpr int GPL = TPL / GS;  // groups per row
        for (int k = 0; k < GPL; ++k) v += sc[(c * GPL + k) * NMU + q];
      } else if constexpr (SHFL) {
        for (int w = 0; w < NT / 64; ++w) v += sc[(w * LN + c) * NMU + q];
      } else {
        for (int k = c; k < NT; k += LN) v += sc[k * NMU + q];
      }
      mus[c * NMU + q] = v;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < LN * kNMom; t += NT) {
      const int c = t / kNMom, q = t % kNMom;
      const int line = tile * LN + c;
      const c64 d = combine_one(mus + c * NMU, fixed(line), q, b, line);
      colv[c * NV + 2 * q] = d.re;
      colv[c * NV + 2 * q + 1] = d.im;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < NV; q += NT) {
      double t = 0.0;
      for (int c = 0; c < LN; ++c) t += colv[c * NV + q];
      dst[(size_t)q * ntiles] = t;
    }
  }
};

// IFFT_cols(in) and the moments of the result (second pass of F^{-1} S; nothing is stored)
template <typename T, int N>
struct OpColsInvMoments : MomentsBase<T, N, false, Ept<T, N>::MOMENT_COLS> {
  static constexpr int DIR1 = +1;
  static constexpr bool TWO = false;
  static constexpr bool ROLLED = true;
  using Acc = typename MomentsBase<T, N, false, Ept<T, N>::MOMENT_COLS>::Acc;
  DBAR_D cx<T> load(int b, int col, int pos) const { return this->inp(b)[(size_t)pos * N + col]; }
  DBAR_D void store(Acc& acc, int b, int col, int pos, cx<T> v) const { this->add(acc, b, col, pos, v); }
};

// x-space operator, first launch: the moments of the input s as it is read, then out = FFT_rows(s) (first pass of
// F s).  With upd_coef set it first updates s by a combination of basis vectors, s -= upd_sign sum_i coef_i V_i over
// upd_nv of them (FP64 accumulation, as the vector kernels; V in FP32 if upd_v32), and stores s back in place: the
// Gram-Schmidt step that produced s (with its |s|^2 partials in upd_part[b][tile]), or the solution update
// x += sum y_i V_i of a cycle end (upd_sign -1) -- the operator's first launch reads s anyway.
// OWN: the update's coefficients are formed by the launch itself (CoefReq), a kernel of its own: its registers cost a full
// batch 8 percent
template <typename T, int N, bool OWN = false>
struct OpRowsFwdMoments : MomentsBase<T, N, true, Ept<T, N>::FWD_MOMENTS> {
  using G = LineGeom<N, Ept<T, N>::FWD_MOMENTS>;
  static constexpr int DIR1 = -1;
  static constexpr bool TWO = false;
  static constexpr bool LOADACC = true;
  static constexpr bool BOXED = true;
  static constexpr bool PRE = true;
  using Pre = Box<N>;
  using Acc = typename MomentsBase<T, N, true, Ept<T, N>::FWD_MOMENTS>::Acc;
  DBAR_D void prologue(int b, Pre& p) const { p = entry_box<N>(this->a, b); }
  static constexpr bool OWN_COEF = OWN;
  // coef_{lo + i} = sigma^2 <v_{lo + i}, w> as ctl_coef_entry forms it (every wave for itself)
  DBAR_D static double own_coef(const CoefReq& o, int b, int i) {
    const double sg = o.ctl[b].sigma[o.lo + i];
    const double h = wave_reduce(o.part + ((size_t)b * o.nval + i) * o.span.stride, o.span.count(b));
    return sg * sg * h;
  }
  DBAR_D cx<T> load(int b, int row, int pos, const Pre& p) const {
    return box_load<T>(entry_rsrc<T, N>(this->inp(b)), row * N + pos, p.col(pos));
  }
  template <int NT>
  DBAR_D void loaded(Acc& acc, int b, int row, int jt, cx<T>* v, int slot, int ntiles, double* scratch,
                     const Pre& p) const {
    const LineArgs& a = this->a;
    if (a.upd_coef) {
      const double* coef = a.upd_coef + (size_t)b * a.upd_coef_bs;
      const int own_lo = OWN && a.own.full && !a.own.full[b] ? a.own.skip : 0;  // (the entry's own window)
      c64 w[G::RMAX];
#pragma unroll
      for (int s = 0; s < G::RMAX; ++s) w[s] = a.upd_zero ? c64{0.0, 0.0} : cvt<double>(v[s]);
#pragma unroll 1
      for (int i = 0; i < a.upd_nv; ++i) {
        double c = 0.0;
        if constexpr (!OWN) c = a.upd_sign * coef[i];
        else if (i >= own_lo) c = own_coef(a.own, b, i);
        if (c == 0.0) continue;  // also keeps never-written basis slots (any bit pattern) out of the sum
        if (sizeof(T) == 8 && a.upd_v32) {
          const Rsrc Vi = entry_rsrc<float, N>(static_cast<const c32*>(a.dotV) + (size_t)b * a.dotV_bs +
                                               (size_t)i * N * N);
#pragma unroll
          for (int s = 0; s < G::RMAX; ++s) {
            const int pos = jt + s * G::TPL;
            w[s] = w[s] - c * cvt<double>(box_load<float>(Vi, row * N + pos, p.col(pos)));
          }
        } else {
          const Rsrc Vi = entry_rsrc<T, N>(static_cast<const cx<T>*>(a.dotV) + (size_t)b * a.dotV_bs +
                                           (size_t)i * N * N);
#pragma unroll
          for (int s = 0; s < G::RMAX; ++s) {
            const int pos = jt + s * G::TPL;
            w[s] = w[s] - c * cvt<double>(box_load<T>(Vi, row * N + pos, p.col(pos)));
          }
        }
      }
      const Rsrc out = entry_rsrc<T, N>(static_cast<const cx<T>*>(a.upd_out) + (size_t)b * a.in_bs);
      double nrm[1] = {0.0};
#pragma unroll
      for (int s = 0; s < G::RMAX; ++s) {
        const int pos = jt + s * G::TPL;
        v[s] = cvt<T>(w[s]);
        box_store<T>(out, row * N + pos, p.col(pos), v[s]);
        nrm[0] += rdot(v[s], v[s]);
      }
      if (a.upd_part) {
        block_reduce_store<NT, 1>(nrm, a.upd_part + (size_t)b * ntiles + slot, 0, scratch);
        __syncthreads();  // the scratch aliases the LDS the transform's first exchange writes
      }
    }
    this->add_loaded(acc, b, row, jt, v);
  }
  DBAR_D void store(Acc&, int b, int row, int pos, cx<T> v, const Pre&) const {
    this->outp(b)[t_index<T, N>(row, pos)] = v;
  }
};

// sum_{n <= MM} c_n w^n by Horner's rule
template <int MM>
DBAR_D c64 g_poly(const c64* __restrict__ c, c64 w) {
  c64 g = c[MM];
#pragma unroll
  for (int n = MM - 1; n >= 0; --n) g = cfma(w, g, c[n]);
  return g;
}
// the same in FP32, from the FP32 roundings of the coefficients
template <int MM>
DBAR_D c32 g_poly32(const c64* __restrict__ c, c32 w) {
  c32 g = cvt<float>(c[MM]);
#pragma unroll
  for (int n = MM - 1; n >= 0; --n) g = cfma(w, g, cvt<float>(c[n]));
  return g;
}

// Per-entry data of the regularised division: the grid offsets (o1, o2) of the regularisation point a and the entry's
// coefficients c_0..c_kMaxM of G (R(0) in slot kMaxM+1), read where they are used: only the points near a need them
// (|xi - a|^2 < 740: 5% of the grid at N = 1024, L = 5), so they are not held in registers across a block's loop.
struct RegPre {
  int o1, o2;
  const c64* c;
};
DBAR_D void regularised_pre(const LineArgs& a, int b, RegPre& p) {
  p.o1 = a.shv ? a.shv[2 * b] : 0;
  p.o2 = a.shv ? a.shv[2 * b + 1] : 0;
  p.c = a.coefG + (size_t)b * kNMom;
}

// R = (S - G)/xi (R(0) from coefG slot kMaxM+1), then out = IFFT_rows(phase * ci * R)
// phase * ci * (S - G)/xi at (row, pos) of entry b, S = sv there (R(0) = coefG slot kMaxM+1 at xi = a)
template <typename T, int N>
DBAR_D cx<T> regularised(const LineArgs& a, const RegPre& p, int row, int pos, cx<T> sv) {
  const c64* c = p.c;
  // xi - a with a = 2i conj(k) on the grid (not reduced modulo the period: the quotient only jumps at the edge),
  // as integer wave numbers: L^2 |xi - a|^2 = m1^2 + m2^2 exactly
  const int m1 = wavenum(pos, N) - p.o1, m2 = wavenum(row, N) - p.o2;
  const int q = m1 * m1 + m2 * m2;
  const double f = ((row + pos) & 1) ? -a.ci : a.ci;
  if (q == 0) return cvt<T>(f * c[kMaxM + 1]);
  const double invL = 1.0 / a.L;
  if constexpr (sizeof(T) == 8) {
    // G only where e^{-|xi|^2} has not underflowed
    const double xi1 = m1 * invL, xi2 = m2 * invL, r2 = xi1 * xi1 + xi2 * xi2;
    if (r2 < 740.0) {
      // unrolled for the order (c_n = 0 beyond M): the coefficient loads are issued together
      const c64 xib{xi1, -xi2};
      const c64 g = a.M == 11 ? g_poly<11>(c, xib) : g_poly<kMaxM>(c, xib);
      sv = sv - exp(-r2) * g;
    }
    const double ir2 = f / r2;
    return cx<T>{(sv.re * xi1 + sv.im * xi2) * ir2, (sv.im * xi1 - sv.re * xi2) * ir2};
  } else {
    // The FP32 operator (inner solves) forms G in FP32 too: S is already rounded to FP32, and G's rounding is of the
    // same size.  e^{-|xi|^2} is zero in FP32 from |xi|^2 = 104 on, so G is formed inside that disc only (|conj(xi)|^n
    // < 2e11 there, far from FP32 overflow).
    const float il = static_cast<float>(invL);
    const float t1 = static_cast<float>(m1) * il, t2 = static_cast<float>(m2) * il;
    const float r2 = t1 * t1 + t2 * t2;
    if (r2 < 104.0f) {
      const c32 w{t1, -t2};
      const c32 g = a.M == 11 ? g_poly32<11>(c, w) : g_poly32<kMaxM>(c, w);
      sv = sv - exp(-r2) * g;
    }
    const float ir2 = static_cast<float>(f) * recip(r2);
    return cx<T>{(sv.re * t1 + sv.im * t2) * ir2, (sv.im * t1 - sv.re * t2) * ir2};
  }
}

template <typename T, int N>
struct OpRowsInvRegular : OpBase<T, N, Ept<T, N>::ROWS> {
  static constexpr int DIR1 = +1;
  static constexpr bool TWO = false;
  using Acc = NoAcc;
  DBAR_D cx<T> load(int b, int row, int pos) const {
    RegPre p;
    regularised_pre(this->a, b, p);
    return regularised<T, N>(this->a, p, row, pos, this->inp(b)[(size_t)row * N + pos]);
  }
  DBAR_D void store(Acc&, int b, int row, int pos, cx<T> v) const { this->outp(b)[(size_t)row * N + pos] = v; }
};

// x-space operator, second launch: S = cf phase FFT_cols(in) (the second pass of F s; optionally stored to sout),
// R = (S - G)/xi, then out = IFFT_cols(phase ci R), between the two column transforms (rolled through LDS: the FP64
// G terms)
template <typename T, int N>
struct OpColsFwdRegInv : OpBase<T, N, Ept<T, N>::REG_COLS> {
  static constexpr int DIR1 = -1;
  static constexpr bool TWO = true;
  static constexpr bool ROLLED = true;
  using Acc = NoAcc;
  static constexpr bool BOXED = true;
  static constexpr bool PRE = true;
  struct Pre {
    RegPre g;
    Box<N> x;
  };
  DBAR_D void prologue(int b, Pre& p) const {
    regularised_pre(this->a, b, p.g);
    p.x = entry_box<N>(this->a, b);
  }
  DBAR_D cx<T> load(int b, int col, int pos, const Pre& p) const {
    return box_load<T>(entry_rsrc<T, N>(this->inp(b)), t_index<T, N>(pos, col), p.x.row(pos));
  }
  template <class A>
  DBAR_D void mid(int b, int col, int pos, cx<T>& v, const Pre& p) const {
    const T f = static_cast<T>(((col + pos) & 1) ? -this->a.cf : this->a.cf);
    const cx<T> S = f * v;
    if (this->a.sout) (static_cast<cx<T>*>(this->a.sout) + (size_t)b * this->a.sout_bs)[(size_t)pos * N + col] = S;
    v = regularised<T, N>(this->a, p.g, pos, col, S);  // row = xi2 index (pos), position = xi1 index (col)
  }
  DBAR_D void store(Acc&, int b, int col, int pos, cx<T> v, const Pre& p) const {
    box_store<T>(entry_rsrc<T, N>(this->outp(b)), t_index<T, N>(pos, col), this->a.box_full || p.x.row(pos), v);
  }
};

// r = IFFT_cols(in); h = r + tail; [hout = h]; u = q_k conj(h); out = FFT_cols(u)   (TAILONLY: stop after hout)
template <typename T, int N, bool TAILONLY, int E = Ept<T, N>::TAIL_COLS>
struct OpColsInvTail : OpBase<T, N, E> {
  static constexpr int DIR1 = +1;
  static constexpr bool TWO = !TAILONLY;
  static constexpr bool ROLLED = true;
  using Acc = NoAcc;
  // (h alone, once per call, keeps the series: its launch gains nothing from the table)
  static constexpr bool TABLE = !TAILONLY && N <= kTailTabMaxN;
  DBAR_D cx<T> load(int b, int col, int pos) const { return this->inp(b)[(size_t)pos * N + col]; }
  DBAR_D cx<T> phase(int b, int col, int pos) const {
    // tabulated in FP64 (arguments up to hundreds of radians; the FP32 operator reads their FP32 roundings); the
    // product is formed in T
    const size_t o = (size_t)b * this->a.e_bs;
    if constexpr (sizeof(T) == 8) return this->a.ex[o + col] * this->a.ey[o + pos];
    else return this->a.ex32[o + col] * this->a.ey32[o + pos];
  }
  // the moments d_0..d_kMaxM of this entry (zero beyond M) in registers, in the transform's precision
  static constexpr bool PRE = true;
  struct Pre {
    cx<T> d[kMaxM + 1];
  };
  DBAR_D void prologue(int b, Pre& p) const {
    const cx<T>* d;
    if constexpr (sizeof(T) == 8) d = this->a.dmom + (size_t)b * kNMom;
    else d = this->a.dmom32 + (size_t)b * kNMom;
#pragma unroll
    for (int n = 0; n <= kMaxM; ++n) p.d[n] = d[n];
  }
  // h = F^{-1}R + sum d_n omega_n; with the shifted regularisation the closed-form part is e^{i a.x} sum d_n omega_n
  DBAR_D cx<T> h_at(int b, int col, int pos, cx<T> v, const Pre& p) const {
    const T x = xgrid_t<T, N>(col, this->a.L), y = xgrid_t<T, N>(pos, this->a.L);
    cx<T> t;
    if constexpr (TABLE) {
      const cx<T> e = static_cast<const cx<T>*>(this->a.ttab)[tail_index<N>(pos, col)];
      t = this->a.M == 11 ? tail_tab<T, 11>(x, y, p.d, e) : tail_tab<T, kMaxM>(x, y, p.d, e);
    } else {
      t = this->a.M == 11 ? tail_sum<T, 11>(x, y, p.d) : tail_sum<T, kMaxM>(x, y, p.d);
    }
    return this->a.shv ? v + conj(phase(b, col, pos)) * t : v + t;
  }
  template <class A>
  DBAR_D void mid(int b, int col, int pos, cx<T>& v, const Pre& p) const {
    const cx<T> h = h_at(b, col, pos, v, p);
    if (this->a.hout) (static_cast<cx<T>*>(this->a.hout) + (size_t)b * this->a.hout_bs)[(size_t)pos * N + col] = h;
    const cx<T> q = (static_cast<const cx<T>*>(this->a.Q) + (size_t)b * this->a.Q_bs)[(size_t)pos * N + col];
    // plain: q_k = Q e_k; shifted (the operator H of equation eqh2): Q alone
    v = (this->a.shv ? q : q * phase(b, col, pos)) * conj(h);
  }
  DBAR_D void store(Acc&, int b, int col, int pos, cx<T> v, const Pre& p) const {
    if constexpr (TAILONLY) {
      cx<T> h = h_at(b, col, pos, v, p);
      if (this->a.tail_phase_out) h = phase(b, col, pos) * h;
      cx<T>* dst = static_cast<cx<T>*>(this->a.hout) + (size_t)b * this->a.hout_bs + (size_t)pos * N + col;
      if (this->a.accumulate) h = h + *dst;
      *dst = h;
    } else {
      this->outp(b)[(size_t)pos * N + col] = v;
    }
  }
};

// X = FFT_rows(in); out = alpha S + beta cf phase X + gamma Y; optional |out|^2 partials
template <typename T, int N>
struct OpRowsFwdEpilogue : OpBase<T, N, Ept<T, N>::ROWS> {
  using G = LineGeom<N, Ept<T, N>::ROWS>;
  static constexpr int DIR1 = -1;
  static constexpr bool TWO = false;
  static constexpr bool DOTS = true;
  struct Acc {
    double v[1];
    double sdot;  // Re<S, out> over this thread's elements (S is the last vector of the fused products)
  };
  DBAR_D cx<T> load(int b, int row, int pos) const { return this->inp(b)[(size_t)row * N + pos]; }
  // X (the row transform's output) is replaced by the stored value, for the Gram-Schmidt products below
  DBAR_D void store(Acc& acc, int b, int row, int pos, cx<T>& X) const {
    const LineArgs& a = this->a;
    const size_t idx = (size_t)row * N + pos;
    const double f = ((row + pos) & 1) ? -a.cf : a.cf;
    c64 o = a.beta * (f * cvt<double>(X));
    c64 sv{0.0, 0.0};
    if (a.alpha != 0.0) {
      sv = cvt<double>((static_cast<const cx<T>*>(a.S) + (size_t)b * a.S_bs)[idx]);
      o = o + a.alpha * sv;
    }
    if (a.gamma != 0.0) o = o + a.gamma * cvt<double>((static_cast<const cx<T>*>(a.Y) + (size_t)b * a.Y_bs)[idx]);
    const cx<T> ot = cvt<T>(o);
    this->outp(b)[idx] = ot;
    X = ot;
    const c64 od = cvt<double>(ot);
    acc.v[0] += norm2(od);
    acc.sdot += sv.re * od.re + sv.im * od.im;
  }
  template <int NT>
  DBAR_D void finish(Acc& acc, int b, int, int slot, int ntiles, double* scratch) const {
    if (!this->a.want_norm) return;
    block_reduce_store<NT, 1>(acc.v, this->a.part + (size_t)b * ntiles + slot, 0, scratch);
  }
  // Re<V_i, out> over this tile for i < dot_nv, from the output values in registers (FP64 accumulation, the order
  // fixed): the multi-dot of the first classical Gram-Schmidt pass without reading the new vector back.  The last
  // vector, V_{dot_nv - 1}, is the epilogue's S (the operator's input) and was accumulated by the stores.
  template <int NT>
  DBAR_D void dots(const Acc& acc, const cx<T>* v, int b, int row, int jt, int tile, int ntiles,
                   double* scratch) const {
    const LineArgs& a = this->a;
    if (a.dot_nv <= 0) return;
    const cx<T>* V = static_cast<const cx<T>*>(a.dotV) + (size_t)b * a.dotV_bs + (size_t)row * N;
    double* dst = a.dot_part + (size_t)b * a.dot_nv * ntiles + tile;
    const double last[1] = {acc.sdot};
    block_reduce_store<NT, 1>(last, dst + (size_t)(a.dot_nv - 1) * ntiles, 0, scratch);
#pragma unroll 1
    for (int i = 0; i < a.dot_nv - 1; ++i) {
      const cx<T>* Vi = V + (size_t)i * N * N;
      double p4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < G::RMAX; ++s) {
        const c64 x = cvt<double>(Vi[jt + s * G::TPL]);
        const c64 w = cvt<double>(v[s]);
        p4[s & 3] += x.re * w.re + x.im * w.im;
      }
      const double val[1] = {(p4[0] + p4[1]) + (p4[2] + p4[3])};
      block_reduce_store<NT, 1>(val, dst + (size_t)i * ntiles, 0, scratch);
    }
  }
};

// x-space operator, third launch: r = IFFT_rows(in) (second pass of F^{-1} R), h = r + sum d_n omega_n, and the
// x-space form of A: out = alpha s + beta q_k conj(h) + gamma Y (F^{-1} of S + i F(q_k conj(h)) is s + i q_k conj(h));
// optional |out|^2 partials, h itself (hout) and the products Re<V_i, out> of the first Gram-Schmidt pass.
// Rows keep every global access of the epilogue and the products contiguous across a wave.
template <typename T, int N>
struct OpRowsInvTailEpi : OpColsInvTail<T, N, false, Ept<T, N>::TAIL_ROWS> {
  using Base = OpColsInvTail<T, N, false, Ept<T, N>::TAIL_ROWS>;
  using G = LineGeom<N, Ept<T, N>::TAIL_ROWS>;
  static constexpr int DIR1 = +1;
  static constexpr bool TWO = false;
  static constexpr bool ROLLED = true;
  static constexpr bool DOTS = true;
  // q_k's potential is one array for the batch: tile-major at N = 4096, where the potential (134 MB in FP32) is
  // otherwise fetched again for most entries (measured 3-7% off the launch); at N = 1024 the tile-major order
  // measured 2-4% slower per launch, and the entry-major order stays
  static constexpr bool TILE_MAJOR = N >= 4096;
  static constexpr bool BOXED = true;
  struct Pre : Base::Pre {
    Box<N> x;
  };
  DBAR_D void prologue(int b, Pre& p) const {
    Base::prologue(b, p);
    p.x = entry_box<N>(this->a, b);
  }
  struct Acc {
    double v[1];
    double sdot;  // Re<S, out> over this thread's elements (S is the last vector of the fused products)
  };
  DBAR_D cx<T> load(int b, int row, int pos, const Pre&) const { return this->inp(b)[t_index<T, N>(row, pos)]; }
  // The stores run GROUP elements at a time: the group's global reads (q, the x factor of e_k, S, Y) are issued
  // together ahead of its tails.  The LDS slot of each element (the row transform's output r) is replaced by the
  // stored value, for the Gram-Schmidt products (zero outside the box).
  // four at a time: wider groups hold more registers than the loads in flight repay (the FP32 launch drops to three
  // waves per SIMD at eight)
  static constexpr int GROUP_W = 4;
  static constexpr int GROUP = G::RMAX < GROUP_W ? G::RMAX : GROUP_W;
  static constexpr bool TABLE = N <= kTailTabMaxN;  // (read with the group)
  struct GroupIn {
    cx<T> q[GROUP], s[GROUP], y[GROUP], ex[GROUP], tab[GROUP];
  };
  // the group's q (times the x factor of e_k on the plain operator), S and Y (zero outside the box)
  DBAR_D void group_load(GroupIn& g, int b, int row, int jt, int s0, const bool (&in)[GROUP]) const {
    const LineArgs& a = this->a;
    const Rsrc Qb = entry_rsrc<T, N>(static_cast<const cx<T>*>(a.Q) + (size_t)b * a.Q_bs);
    const Rsrc Sb = entry_rsrc<T, N>(static_cast<const cx<T>*>(a.S) + (size_t)b * a.S_bs);
    const Rsrc Yb = entry_rsrc<T, N>(static_cast<const cx<T>*>(a.Y) + (size_t)b * a.Y_bs);
    const size_t eo = (size_t)b * a.e_bs;
#pragma unroll
    for (int u = 0; u < GROUP; ++u) {
      const int pos = jt + (s0 + u) * G::TPL;
      const uint32_t idx = row * N + pos;
      g.q[u] = box_load<T>(Qb, idx, in[u]);
      g.s[u] = a.alpha != 0.0 ? box_load<T>(Sb, idx, in[u]) : cx<T>{T(0), T(0)};
      if constexpr (TABLE) g.tab[u] = static_cast<const cx<T>*>(a.ttab)[tail_index<N>(row, pos)];
      g.y[u] = (a.gamma != 0.0 && !a.y_rhs) ? box_load<T>(Yb, idx, in[u]) : cx<T>{T(0), T(0)};
      if (a.shv) g.ex[u] = cx<T>{T(1), T(0)};
      else if constexpr (sizeof(T) == 8) g.ex[u] = a.ex[eo + pos];
      else g.ex[u] = a.ex32[eo + pos];
    }
  }
  template <int LS>
  DBAR_D void store_all(Acc& acc, int b, int row, int jt, cx<T>* my, const Pre& p) const {
    static_assert(G::RMAX % GROUP == 0, "whole groups");
    const LineArgs& a = this->a;
    const size_t base = (size_t)row * N;
    // the y factor of e_k is the row's (1 with the shifted regularisation, where q stands alone)
    cx<T> ey{T(1), T(0)};
    if (!a.shv) {
      if constexpr (sizeof(T) == 8) ey = a.ey[(size_t)b * a.e_bs + row];
      else ey = a.ey32[(size_t)b * a.e_bs + row];
    }
    const bool row_in = p.x.row(row);
    const Rsrc outb = entry_rsrc<T, N>(this->outp(b));
    const Rsrc out32 = entry_rsrc<float, N>(static_cast<const c32*>(a.out32) + (size_t)b * a.out32_bs);
#pragma unroll 1
    for (int s0 = 0; s0 < G::RMAX; s0 += GROUP) {
      bool in[GROUP];
#pragma unroll
      for (int u = 0; u < GROUP; ++u) in[u] = row_in && p.x.col(jt + (s0 + u) * G::TPL);
      GroupIn cur;
      group_load(cur, b, row, jt, s0, in);
#pragma unroll
      for (int u = 0; u < GROUP; ++u) {
        const int pos = jt + (s0 + u) * G::TPL;
        cx<T>& slot = my[G::padded(pos) * LS];
        if (!in[u] && !a.hout) {  // outside the box only h is formed
          slot = cx<T>{T(0), T(0)};
          continue;
        }
        cx<T> h;
        if constexpr (TABLE) {
          const T x = xgrid_t<T, N>(pos, a.L), y = xgrid_t<T, N>(row, a.L);
          const cx<T> t = a.M == 11 ? tail_tab<T, 11>(x, y, p.d, cur.tab[u]) : tail_tab<T, kMaxM>(x, y, p.d, cur.tab[u]);
          h = a.shv ? slot + conj(this->phase(b, pos, row)) * t : slot + t;
        } else {
          h = this->h_at(b, pos, row, slot, p);  // x index pos, y index row
        }
        if (a.hout) (static_cast<cx<T>*>(a.hout) + (size_t)b * a.hout_bs)[base + pos] = h;
        const cx<T> qk = cur.q[u] * (cur.ex[u] * ey);
        const cx<T> w = qk * conj(h);
        const cx<T> yv = a.y_rhs ? mul_mi(qk) : cur.y[u];
        cx<T> ot;
        if constexpr (sizeof(T) == 8) {
          ot = a.beta * w + a.alpha * cur.s[u] + a.gamma * yv;
        } else {  // the FP32 operator's result is FP32: form it in FP32
          ot = cvt<T>(a.beta) * w + static_cast<T>(a.alpha) * cur.s[u] + static_cast<T>(a.gamma) * yv;
        }
        if (!in[u]) ot = cx<T>{T(0), T(0)};  // (q is zero there, but h may not be finite)
        const uint32_t idx = row * N + pos;
        if (a.out) box_store<T>(outb, idx, in[u], ot);
        if constexpr (sizeof(T) == 8) {
          if (a.out32) box_store<float>(out32, idx, in[u], cvt<float>(ot));
        }
        slot = ot;
        acc.v[0] += rdot(ot, ot);
        acc.sdot += rdot(cur.s[u], ot);
      }
    }
  }
  template <int NT>
  DBAR_D void finish(Acc& acc, int b, int, int slot, int ntiles, double* scratch) const {
    if (!this->a.want_norm) return;
    block_reduce_store<NT, 1>(acc.v, this->a.part + (size_t)b * ntiles + slot, 0, scratch);
  }
  // Re<V_i, out> over this tile for i < dot_nv (FP64 accumulation, the order fixed); V_{dot_nv - 1} is S, whose
  // products the stores accumulated, as they did |out|^2 (value dot_nv with dot_self).  Each wave reduces its
  // products by shuffles and parks them in LDS; one barrier
  // then serves all of them (the waves read their next V_i while others still compute).
  template <int NT>
  DBAR_D void dots(const Acc& acc, const cx<T>* v, int b, int row, int jt, int tile, int ntiles,
                   double* scratch, const Pre& p) const {
    const LineArgs& a = this->a;
    const int nv = a.dot_nv;
    if (nv <= 0) return;
    const int nval = nv + (a.dot_self ? 1 : 0);
    // vectors below the entry's Gram-Schmidt window (never V_{nv - 1}, the input itself)
    const int skip = (a.dot_full && !a.dot_full[b]) ? a.dot_skip : 0;
    const cx<T>* V = static_cast<const cx<T>*>(a.dotV) + (size_t)b * a.dotV_bs;
    double* dst = a.dot_part + (size_t)b * nval * ntiles + tile;
    const bool row_in = p.x.row(row);
    auto partial = [&](int i) {
      const Rsrc Vi = entry_rsrc<T, N>(V + (size_t)i * N * N);
      double p4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < G::RMAX; ++s) {
        const int pos = jt + s * G::TPL;
        p4[s & 3] += rdot(box_load<T>(Vi, row * N + pos, row_in && p.x.col(pos)), v[s]);
      }
      return (p4[0] + p4[1]) + (p4[2] + p4[3]);
    };
    if constexpr (NT >= 64) {
      constexpr int NW = NT / 64;
      const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
      __syncthreads();  // scratch aliases the LDS the stores and the norm reduction used
      double x = wsum(acc.sdot);
      if (lane == 0) scratch[(nv - 1) * NW + wave] = x;
      if (a.dot_self) {
        x = wsum(acc.v[0]);
        if (lane == 0) scratch[nv * NW + wave] = x;
      }
#pragma unroll 1
      for (int i = 0; i < nv - 1; ++i) {
        x = i < skip ? 0.0 : wsum(partial(i));
        if (lane == 0) scratch[i * NW + wave] = x;
      }
      __syncthreads();
      for (int i = threadIdx.x; i < nval; i += NT) {
        double t = 0.0;
        for (int q = 0; q < NW; ++q) t += scratch[i * NW + q];
        dst[(size_t)i * ntiles] = t;
      }
    } else {
      const double last[1] = {acc.sdot};
      block_reduce_store<NT, 1>(last, dst + (size_t)(nv - 1) * ntiles, 0, scratch);
      if (a.dot_self) block_reduce_store<NT, 1>(acc.v, dst + (size_t)nv * ntiles, 0, scratch);
#pragma unroll 1
      for (int i = 0; i < nv - 1; ++i) {
        const double val[1] = {i < skip ? 0.0 : partial(i)};
        block_reduce_store<NT, 1>(val, dst + (size_t)i * ntiles, 0, scratch);
      }
    }
  }
};

// out = FFT_cols(Q e_k)
template <typename T, int N>
struct OpColsFwdPotential : OpBase<T, N, Ept<T, N>::COLS> {
  static constexpr int DIR1 = -1;
  static constexpr bool TWO = false;
  using Acc = NoAcc;
  DBAR_D cx<T> load(int b, int col, int pos) const {
    const c64 q = cvt<double>((static_cast<const cx<T>*>(this->a.Q) + (size_t)b * this->a.Q_bs)[(size_t)pos * N + col]);
    const c64 e = this->a.ex[(size_t)b * this->a.e_bs + col] * this->a.ey[(size_t)b * this->a.e_bs + pos];
    return cvt<T>(q * e);
  }
  DBAR_D void store(Acc&, int b, int col, int pos, cx<T> v) const { this->outp(b)[(size_t)pos * N + col] = v; }
};

// out = FFT_cols(in) (DIR -1) or IFFT_cols(in) (DIR +1)
template <typename T, int N, int DIR>
struct OpColsPlain : OpBase<T, N, Ept<T, N>::COLS> {
  static constexpr int DIR1 = DIR;
  static constexpr bool TWO = false;
  using Acc = NoAcc;
  DBAR_D cx<T> load(int b, int col, int pos) const { return this->inp(b)[(size_t)pos * N + col]; }
  DBAR_D void store(Acc&, int b, int col, int pos, cx<T> v) const { this->outp(b)[(size_t)pos * N + col] = v; }
};

// ------------------------------------------------------------------------------------------------------------
// The generic line kernel
// ------------------------------------------------------------------------------------------------------------
DBAR_D int xcd_swizzle(int bid, int nblk) {
  // blocks are dispatched round-robin over the 8 XCDs; give each XCD a contiguous range of tiles so that tiles
  // sharing cache lines (narrow column tiles) meet in the same L2
  if ((nblk & 7) != 0) return bid;
  return (bid & 7) * (nblk >> 3) + (bid >> 3);
}


// Boxed row launches with at least this many tiles give each XCD a contiguous range of them; with fewer, consecutive
// blocks (tiles, then entries) simply go round the XCDs, which keeps all of them busy however few tiles a box has.
constexpr int kSpreadTiles = 128;

// Occupancy floor: at least 4 waves per SIMD (<= 128 VGPRs) for the wide column tiles, whose LDS allows two
// blocks per CU only if the registers do too, and for FP32 rows (the tail's reads would take 20 more).
template <int NT, bool COLS, bool MOMENTS, bool FP32>
struct MinWaves {
  static constexpr int value = COLS && NT >= 256 ? (MOMENTS ? NT / 256 : 4) : !COLS && FP32 ? 4 : 1;
};

template <typename T, int N, int LINES, bool COLS, class Op>
__global__ void __launch_bounds__((LINES * Op::G::TPL), (MinWaves<LINES * Op::G::TPL, COLS, Op::MOMENTS, sizeof(T) == 4>::value))
    k_lines(Op op) {
  using G = typename Op::G;
  constexpr int NT = LINES * G::TPL;
  __shared__ cx<T> lds[LdsSize<T, G, LINES, COLS, Op::MOMENTS>::kElems];
  // pass-1 twiddle table: column stages only (their element work makes them arithmetic-bound)
  __shared__ cx<T> lds_t1[COLS ? Pass1Table<G>::SIZE : 1];
  constexpr int NTILES = N / LINES;
  int b, tile, slot;
  if constexpr (Op::BOXED && !COLS) {
    // rows of the entry's box only: its cnt tiles from t0 on, partials in slots 0 .. cnt - 1; the launch covers the
    // largest box of the batch.  With many tiles, block i of an entry goes to XCD i mod 8, which takes a contiguous
    // eighth of them (neighbouring tiles share lines of the tiled array).  TILE_MAJOR: the entries of a tile follow one
    // another on its XCD, i / 8 = (tile's place on the XCD) * entries + entry.
    constexpr bool SPREAD = NTILES >= kSpreadTiles;
    static_assert(SPREAD || !Op::TILE_MAJOR, "tile-major launches spread their tiles over the XCDs");
    int k = SPREAD ? blockIdx.x >> 3 : blockIdx.x;
    if constexpr (Op::TILE_MAJOR) {
      const int nb = op.a.B;
      b = k % nb;
      k /= nb;
    } else {
      b = blockIdx.y;
      if constexpr (Op::OWN_COEF) {
        // The blocks beyond the entries take the step's coefficients to its record and decide on its end, beside the
        // update.  An entry that ends there may still be updated and transformed by blocks that read its flag before
        // (a whole block at a time: block_flag): nothing uses what they write (the flag is off for every later launch of
        // the cycle).
        if (b >= op.a.B) {
          const CoefReq& o = op.a.own;
          static_assert(NT >= 64, "whole waves");
          if (blockIdx.x < op.a.B && o.act[blockIdx.x])
            ctl_coef_entry(blockIdx.x, o.ctl, o.part, o.nval, o.span, o.act, o.fs, o.j, 0, 1, o.m, o.lo, o.skip, o.full);
          return;
        }
      }
    }
    if constexpr (Op::OWN_COEF) {
      if (!block_flag(op.a.act + b)) return;
    } else {
      if (!op.active(b)) return;
    }
    int t0 = 0, cnt = NTILES;
    if (N >= kBoxMinN && op.a.box && !op.a.box_full) {
      const Box<N> x = entry_box<N>(op.a, b);
      t0 = x.r0 / LINES;
      cnt = x.r1 / LINES - t0;
    }
    slot = k;
    if constexpr (SPREAD) {
      const int per = (cnt + 7) >> 3;
      slot = (blockIdx.x & 7) * per + k;
      if (k >= per) return;
    }
    if (slot >= cnt) return;
    tile = t0 + slot;
  } else {
    b = blockIdx.y;
    tile = slot = xcd_swizzle(blockIdx.x, gridDim.x);
    if (!op.active(b)) return;
  }
  typename Op::Pre pre;
  op.prologue(b, pre);
  const int tid = threadIdx.x;
  const int ln = COLS ? (tid % LINES) : (tid / G::TPL);
  const int jt = COLS ? (tid / LINES) : (tid % G::TPL);
  const int line = tile * LINES + ln;
  const cx<T>* tw = static_cast<const cx<T>*>(op.a.tw);
  if constexpr (COLS) fill_pass1_table<T, G>(lds_t1, tw, tid, NT);

  typename Op::Acc acc{};
  cx<T> v[G::RMAX];
#pragma unroll
  for (int s = 0; s < G::RMAX; ++s) {
    if constexpr (Op::BOXED) v[s] = op.load(b, line, jt + s * G::TPL, pre);
    else v[s] = op.load(b, line, jt + s * G::TPL);
  }
  if constexpr (Op::LOADACC)
    op.template loaded<NT>(acc, b, line, jt, v, slot, NTILES, reinterpret_cast<double*>(lds), pre);
  // LDS: a row tile keeps each line contiguous (one line per wave or less); a column tile interleaves its lines
  // element by element, so that the lanes of a wave (consecutive columns) hit consecutive banks
  constexpr int LS = COLS ? LINES : 1;
  cx<T>* my = COLS ? lds + ln : lds + ln * G::LDS_LINE;
  line_fft<T, G, Op::DIR1, LS, COLS>(v, jt, my, tw, lds_t1);
  // Heavy per-element work (FP64 moments, the closed-form tail) runs in a rolled loop over values parked in LDS at
  // the thread's own positions: registers stay low (occupancy) and no barrier is needed until the next exchange.
  if constexpr (Op::TWO) {
    if constexpr (Op::ROLLED) {
#pragma unroll
      for (int s = 0; s < G::RMAX; ++s) my[G::padded(jt + s * G::TPL) * LS] = v[s];
#pragma unroll 1
      for (int s = 0; s < G::RMAX; ++s) {
        const int pos = jt + s * G::TPL;
        cx<T> t = my[G::padded(pos) * LS];
        if constexpr (Op::PRE) op.template mid<typename Op::Acc>(b, line, pos, t, pre);
        else op.template mid<typename Op::Acc>(b, line, pos, t);
        my[G::padded(pos) * LS] = t;
      }
#pragma unroll
      for (int s = 0; s < G::RMAX; ++s) v[s] = my[G::padded(jt + s * G::TPL) * LS];
      __syncthreads();  // the forward transform's first exchange writes other threads' positions
    } else {
#pragma unroll
      for (int s = 0; s < G::RMAX; ++s) {
        if constexpr (Op::PRE) op.template mid<typename Op::Acc>(b, line, jt + s * G::TPL, v[s], pre);
        else op.template mid<typename Op::Acc>(b, line, jt + s * G::TPL, v[s]);
      }
    }
    line_fft<T, G, -Op::DIR1, LS, COLS>(v, jt, my, tw, lds_t1);
  }
  if constexpr (Op::ROLLED && !Op::TWO) {
#pragma unroll
    for (int s = 0; s < G::RMAX; ++s) my[G::padded(jt + s * G::TPL) * LS] = v[s];
    if constexpr (Op::GROUP > 1) {
      op.template store_all<LS>(acc, b, line, jt, my, pre);
    } else {
#pragma unroll 1
      for (int s = 0; s < G::RMAX; ++s) {
        const int pos = jt + s * G::TPL;
        if constexpr (Op::PRE) op.store(acc, b, line, pos, my[G::padded(pos) * LS], pre);
        else op.store(acc, b, line, pos, my[G::padded(pos) * LS]);
      }
    }
    // the stored values (the stores may replace them) back to registers for the products below, before the
    // reductions reuse the LDS (the thread's own positions: no barrier)
    if constexpr (Op::DOTS) {
#pragma unroll
      for (int s = 0; s < G::RMAX; ++s) v[s] = my[G::padded(jt + s * G::TPL) * LS];
    }
  } else {
#pragma unroll
    for (int s = 0; s < G::RMAX; ++s) {
      if constexpr (Op::PRE) op.store(acc, b, line, jt + s * G::TPL, v[s], pre);
      else op.store(acc, b, line, jt + s * G::TPL, v[s]);
    }
  }
  op.template finish<NT>(acc, b, tile, slot, NTILES, reinterpret_cast<double*>(lds));
  if constexpr (Op::DOTS && Op::BOXED)
    op.template dots<NT>(acc, v, b, line, jt, slot, NTILES, reinterpret_cast<double*>(lds), pre);
  else if constexpr (Op::DOTS)
    op.template dots<NT>(acc, v, b, line, jt, slot, NTILES, reinterpret_cast<double*>(lds));
}

template <typename T, int N, bool COLS, class Op, int V = 0>
void launch_op(const LineArgs& a, hipStream_t s) {
  constexpr int LINES = COLS ? Tiling<T, N>::template cols_of<Op::G::RMAX, V, Op::MOMENTS>() : Tiling<T, N>::ROWS;
  constexpr int NT = LINES * Op::G::TPL;
  Op op;
  op.a = a;
  int tiles = N / LINES;
  if constexpr (Op::BOXED && !COLS) {
    // the tiles of the largest box, rounded up to a sixteenth of the grid (captured graphs are kept per launch size):
    // whole rounds of the eight XCDs where the tiles are spread over them
    constexpr int STEP = N / LINES > 16 ? N / LINES / 16 : 1;
    static_assert(N / LINES < kSpreadTiles || STEP % 8 == 0, "whole rounds");
    if (a.box && !a.box_full) tiles = (a.box_rows / LINES + STEP - 1) / STEP * STEP;
  }
  const dim3 grid = Op::TILE_MAJOR ? dim3(tiles * a.B) : dim3(tiles, a.B + (Op::OWN_COEF ? 1 : 0));
  hipLaunchKernelGGL((k_lines<T, N, LINES, COLS, Op>), grid, dim3(NT), 0, s, op);
}

// column stages at tile variant V (only the valid variants are instantiated)
template <typename T, int N, class Op>
void launch_cols(const LineArgs& a, hipStream_t s) {
  if constexpr (Tiling<T, N>::template cols_valid<3>()) {
    if (a.tile == 3) return launch_op<T, N, true, Op, 3>(a, s);
  }
  if constexpr (Tiling<T, N>::template cols_valid<2>()) {
    if (a.tile == 2) return launch_op<T, N, true, Op, 2>(a, s);
  }
  if constexpr (Tiling<T, N>::template cols_valid<1>()) {
    if (a.tile == 1) return launch_op<T, N, true, Op, 1>(a, s);
  }
  launch_op<T, N, true, Op, 0>(a, s);
}

template <typename T, int N>
void launch_lines(LineOp op, const LineArgs& a, hipStream_t s) {
  switch (op) {
    case LineOp::RowsInvScaled: launch_op<T, N, false, OpRowsInvScaled<T, N>>(a, s); break;
    case LineOp::ColsInvMoments: launch_cols<T, N, OpColsInvMoments<T, N>>(a, s); break;
    case LineOp::RowsInvRegular: launch_op<T, N, false, OpRowsInvRegular<T, N>>(a, s); break;
    case LineOp::ColsInvTailFwd: launch_cols<T, N, OpColsInvTail<T, N, false>>(a, s); break;
    case LineOp::ColsInvTail: launch_cols<T, N, OpColsInvTail<T, N, true>>(a, s); break;
    case LineOp::RowsFwdEpilogue: launch_op<T, N, false, OpRowsFwdEpilogue<T, N>>(a, s); break;
    case LineOp::ColsFwdPotential: launch_cols<T, N, OpColsFwdPotential<T, N>>(a, s); break;
    case LineOp::ColsFwdPlain: launch_cols<T, N, OpColsPlain<T, N, -1>>(a, s); break;
    case LineOp::ColsInvPlain: launch_cols<T, N, OpColsPlain<T, N, +1>>(a, s); break;
    case LineOp::RowsFwdMoments:
      if constexpr (N >= 64 && N <= kOwnCoefMaxN) {
        if (a.own.part) {
          launch_op<T, N, false, OpRowsFwdMoments<T, N, true>>(a, s);
          break;
        }
      }
      launch_op<T, N, false, OpRowsFwdMoments<T, N>>(a, s);
      break;
    case LineOp::ColsFwdRegularInv: launch_cols<T, N, OpColsFwdRegInv<T, N>>(a, s); break;
    case LineOp::RowsInvTailEpilogue: launch_op<T, N, false, OpRowsInvTailEpi<T, N>>(a, s); break;
  }
}

#define DBAR_INSTANTIATE_N(NN)                                                  \
  template void launch_lines<double, NN>(LineOp, const LineArgs&, hipStream_t); \
  template void launch_lines<float, NN>(LineOp, const LineArgs&, hipStream_t);

}  // namespace dbar
