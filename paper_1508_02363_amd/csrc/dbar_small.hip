// A whole Krylov cycle of the x-space iteration in one launch, for grids that fit the LDS of one block (N = 16, 32, 64).
//
// On such a grid the three operator launches and the two control launches of a step are a few microseconds of work each
// between launch latencies, and with thousands of entries (the DS II scattering transforms solve one problem per grid
// point) every step moves the transform array through memory four times.  Here one block per entry keeps the transform
// array in LDS and the GMRES record in the registers of its first wave, and runs the steps of the cycle one after the
// other: the operator (moments, row and column transforms, division by xi, inverse transforms, tail), the Gram-Schmidt
// products and update, the Givens step, the convergence test.  Only the basis vectors go to memory.  Steps, windows,
// early convergence decision and restart flags are those of the launch-per-stage cycle (krylov_cycle).
//
// Layout: thread t holds, in the row layout, elements jt + q TPL of row t / TPL (jt = t % TPL) and, in the column layout,
// elements jt + q TPL of column t % N (jt = t / N); the array crosses between them in LDS with a pitch of N + 4 elements
// (rows of one wave then start 16 banks apart).  Eight elements per thread at N = 64 (512 threads, up to 256 VGPRs, one
// block per CU), four below; sixteen waves with four elements each spend more on exchanges and spill (N = 64 FP64).
//
// What bounds it: the chain of a step inside one block, about 55 thousand cycles at N = 64 in FP64 (division with its
// polynomial 10, tail 14, the four transforms and two transposes 13, moments 10, Gram-Schmidt products, decision and update
// 7, Givens 3); LDS and registers allow one block per CU.  Measured, launch per stage -> whole cycle: a potential
// reconstructed on 64^2 (4096 problems) 11.7 -> 6.1 ms, one FP64 problem at N = 64 1.15 -> 0.64 ms, 4096
// problems 20.3 -> 11.3 ms.  N = 128 does not fit one block's LDS.  The previous basis vector stays in LDS (its products
// and its part of the update read it there: 4096 problems 12.3 -> 11.3 ms, what is left of the L2 goes to v_j).
#include "dbar_ctl.h"
#include "dbar_launch.h"
#include "dbar_lines.h"
#include "dbar_solver.h"

namespace dbar {
namespace {

constexpr int kMaxM1 = kMaxM + 1;

template <typename T, int N>
struct SmallGeom {
  static constexpr int E = N == 64 ? 8 : 4;
  using G = LineGeom<N, E>;
  static constexpr int TPL = G::TPL;
  static constexpr int NT = N * TPL;
  static constexpr int NW = NT / 64;
  static constexpr int PITCH = N + 4;
  static constexpr int MU = 2 * (kMaxM + 1);
  static constexpr int NP = (kMaxM + 1) * (kMaxM + 2);  // real sums P_kl, k + l <= kMaxM
  static constexpr size_t kData = (size_t)G::padded(N) * PITCH * sizeof(cx<T>);
  static constexpr size_t kScratch = ((size_t)N * MU + 2 * NP) * sizeof(double);
  static constexpr size_t kBytes = kData > kScratch ? kData : kScratch;
  static_assert(NT % 64 == 0 && NT <= 1024, "whole waves, one block");
  static_assert(N * G::LDS_LINE <= G::padded(N) * PITCH, "the row lines fit the transposed array's space");
};

struct SmallArgs {
  LineArgs first;   // the operator's pass (iterated method: the shifted pass)
  LineArgs second;  // iterated method: the k = 0 pass
  void* V = nullptr;
  size_t V_bs = 0;
  Ctl* ctl = nullptr;
  int* act = nullptr;
  int fs = 0, m = 0, mlim = 0, window = 0;
  double wscale = 0.0;
};

template <typename T, int N>
struct SmallShared {
  alignas(16) unsigned char data[SmallGeom<T, N>::kBytes];
  alignas(16) cx<T> prev[N * N];  // v_{j-1}, row layout, each thread's own elements (element s of thread t at s NT + t)
  c64 coefG[kNMom];
  cx<T> d[kMaxM + 1];
  double ypow[N * (kMaxM + 2)];  // y_row^l
  double binom[kMaxM1 * kMaxM1], invfact[kMaxM1];
  T e1[2][2][N];                 // e^{-(xi - a)^2} of either pass, along xi1 and xi2
  double red[(kMaxRestart + 2) * SmallGeom<T, N>::NW];
  // the GMRES record of the cycle (Ctl's fields of the same names)
  double sigma[kMaxRestart + 1], g[kMaxRestart + 1], cs[kMaxRestart], sn[kMaxRestart], hsum[kMaxRestart],
      coef[kMaxRestart];
  int stop;
};

// Step j's Givens rotation from beta = ||v_{j+1}|| (first wave): the record's next entries and the column of H; returns
// the residual estimate.
template <typename T, int N>
DBAR_D double small_givens(Ctl& c, SmallShared<T, N>& sh, int j, double beta, double top, double mine) {
  const int lane = threadIdx.x & 63;
  const double gj = sh.g[j], sub = sh.sigma[j] * beta, den = hypot(top, sub);
  const double cs = den > 0.0 ? top / den : 1.0, sn = den > 0.0 ? sub / den : 0.0;
  double* col = c.H + (size_t)j * (kMaxRestart + 1);
  if (lane < j) col[lane] = mine;
  if (lane == 0) {
    col[j] = den;
    col[j + 1] = 0.0;
    sh.cs[j] = cs;
    sh.sn[j] = sn;
    sh.g[j] = cs * gj;
    sh.g[j + 1] = -sn * gj;
    sh.sigma[j + 1] = beta > 0.0 ? 1.0 / beta : 0.0;
  }
  return fabs(-sn * gj);
}
// entry j of step j's column after the previous rotations (first wave), and the entries before it, one per lane
template <typename T, int N>
DBAR_D double small_column(const SmallShared<T, N>& sh, int j, double& mine) {
  const int lane = threadIdx.x & 63;
  const HessLane h = hess_lane(lane < j ? sh.cs[lane] : 1.0, lane < j ? sh.sn[lane] : 0.0, sh.sigma[j], j,
                               lane <= j ? sh.hsum[lane] : 0.0);
  return hess_rotate(h, j, mine);
}

// x, opaque to the compiler: what is computed from it in one step of the cycle is not kept in registers for the next
// (hoisted out of the loop over the steps, the positions and table addresses alone would fill them)
DBAR_D int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
// the first lane's value, for values all lanes hold: scalar registers instead of a vector register each
DBAR_D double uniform(double x) {
  const long long v = __builtin_bit_cast(long long, x);
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)v), hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
DBAR_D float uniform(float x) { return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x))); }

// 1/r to about one ulp for r = 0 (infinite, unused) and the normal range: the hardware estimate and two Newton steps
DBAR_D double recip_newton(double r) {
  double y = __builtin_amdgcn_rcp(r);
  y = fmar(y, fmar(-r, y, 1.0), y);
  return fmar(y, fmar(-r, y, 1.0), y);
}

// Moments of s (row layout, v), regularised about the point a.shv names: d_n to sh.d, c_n and R(0) to sh.coefG.  KK: the
// order the sums are unrolled for.
template <typename T, int N, int KK>
DBAR_D void small_moments(const LineArgs& a, int b, const cx<T>* v, int row, int jt, SmallShared<T, N>& sh,
                          double wscale) {
  using S = SmallGeom<T, N>;
  constexpr int NV = 2 * (KK + 1);
  T acc[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) acc[q] = T(0);
#pragma unroll
  for (int s = 0; s < S::E; ++s) {
    const int pos = jt + s * S::TPL;
    cx<T> sv = v[s];
    if (a.shv) {
      const size_t o = (size_t)b * a.e_bs;
      if constexpr (sizeof(T) == 8) sv = sv * (a.ex[o + pos] * a.ey[o + row]);
      else sv = sv * (a.ex32[o + pos] * a.ey32[o + row]);
    }
    const T t = xgrid_t<T, N>(pos, a.L);
    T tp = T(1);
#pragma unroll
    for (int k = 0; k <= KK; ++k) {
      acc[2 * k] += tp * sv.re;
      acc[2 * k + 1] += tp * sv.im;
      tp *= t;
    }
  }
  const int lane = threadIdx.x & 63;
  constexpr int OFF = S::TPL / 2;
  const int base = reduce_lanes<NV, OFF, 1>(acc, lane);
  const bool mine = (lane & reduce_copies<NV, OFF, 1>()) == 0;
  constexpr int KEEP = reduce_left<NV, OFF, 1>();
  double* mu = reinterpret_cast<double*>(sh.data);  // [row][S::MU]
  double* P = mu + N * S::MU;                       // [half of the rows][k, l][re, im]
  __syncthreads();                                  // the data area is free
#pragma unroll
  for (int i = 0; i < KEEP; ++i)
    if (mine) mu[row * S::MU + base + i] = static_cast<double>(acc[i]);
  __syncthreads();
  // P_kl = sum over the rows of y^l mu_k, k + l <= max(M, 1): one thread per real sum and half of the rows.  Then
  // d_n = sum_k C(n, k) i^{n-k} P_k,n-k and the conj moment sum (x - i y) s = P_10 - i P_01 (a binomial expansion per
  // row, as the row launches do it, is sixty-four of them).
  const int top = a.M > 1 ? a.M : 1, nl = top + 1, np = nl * (nl + 1);  // np: reals
  for (int t = threadIdx.x; t < 2 * np; t += S::NT) {
    const int half = t >= np, i = half ? t - np : t, c = i & 1;
    int l = 0, k = i >> 1;
    while (k > top - l) k -= top + 1 - l++;  // pairs ordered by l, then k
    const double* m = mu + half * (N / 2) * S::MU + 2 * k + c;
    const double* yp = sh.ypow + half * (N / 2) * (kMaxM + 2) + l;
    double x0 = 0.0, x1 = 0.0;
#pragma unroll 4
    for (int r = 0; r < N / 2; r += 2) {
      x0 += yp[r * (kMaxM + 2)] * m[r * S::MU];
      x1 += yp[(r + 1) * (kMaxM + 2)] * m[(r + 1) * S::MU];
    }
    P[half * S::NP + i] = x0 + x1;
  }
  __syncthreads();
  // sixteen lanes per Taylor slot, one term each
  const int k = threadIdx.x & 15;
  for (int n = threadIdx.x >> 4; n < kNMom; n += S::NT / 16) {
    c64 p{0.0, 0.0};
    const bool dt = n == kMaxM + 1;  // P_10 - i P_01
    if (dt ? k < 2 : n <= a.M && k <= n) {
      const int l = dt ? 1 - k : n - k, i = 2 * (l * nl - l * (l - 1) / 2 + k);  // (the pairs of smaller l come first)
      p = c64{P[i] + P[S::NP + i], P[i + 1] + P[S::NP + i + 1]};
      if (dt) {
        if (k == 0) p = mul_mi(p);
      } else {
        p = sh.binom[n * kMaxM1 + k] * p;
        const int e = l & 3;  // times i^{n-k}
        p = e == 0 ? p : e == 1 ? mul_i(p) : e == 2 ? -p : mul_mi(p);
      }
    }
    const c64 d{wscale * add_xor<1>(add_xor<2>(add_xor<4>(add_xor<8>(p.re)))),
                wscale * add_xor<1>(add_xor<2>(add_xor<4>(add_xor<8>(p.im))))};
    if (k == 0) {
      if (dt) {
        sh.coefG[n] = c64{0.0, -0.5} * d;
      } else {
        sh.d[n] = cvt<T>(d);
        sh.coefG[n] = taylor_power(n, sh.invfact[n] * d);
      }
    }
  }
  __syncthreads();
}

// v (row layout): s -> F^{-1}((S - G)/(xi - a)) with S = F s; the moments' results stay in sh
template <typename T, int N, int MM, int PASS>
DBAR_D void small_inverse(const LineArgs& a, int b, cx<T>* v, int row, int jt, SmallShared<T, N>& sh, double wscale) {
  using S = SmallGeom<T, N>;
  using G = typename S::G;
  small_moments<T, N, MM>(a, b, v, row, jt, sh, wscale);
  const cx<T>* tw = static_cast<const cx<T>*>(a.tw);
  cx<T>* data = reinterpret_cast<cx<T>*>(sh.data);
  const int tid = fresh(threadIdx.x), col = tid % N, jc = tid / N;
  line_fft<T, G, -1, 1, false>(v, jt, data + row * G::LDS_LINE, tw, nullptr);
#pragma unroll
  for (int s = 0; s < S::E; ++s) data[G::padded(row) * S::PITCH + jt + s * S::TPL] = v[s];
  __syncthreads();
#pragma unroll
  for (int s = 0; s < S::E; ++s) v[s] = data[G::padded(jc + s * S::TPL) * S::PITCH + col];
  __syncthreads();
  line_fft<T, G, -1, S::PITCH, false>(v, jc, data + col, tw, nullptr);
#pragma unroll
  for (int s = 0; s < S::E; ++s) data[G::padded(jc + s * S::TPL) * S::PITCH + col] = v[s];  // the thread's own slots
  // R = (S - G)/(xi - a) as `regularised` forms it, with G's exponential as a product of two table values and the sums in
  // the transform's precision; G counts everywhere (on these grids most points are near a)
  {
    const int o1 = a.shv ? a.shv[2 * b] : 0, o2 = a.shv ? a.shv[2 * b + 1] : 0;
    const T* e1 = sh.e1[PASS][0];
    const T* e2 = sh.e1[PASS][1];
    const T il = static_cast<T>(1.0 / a.L), cf = static_cast<T>(a.cf), ci = static_cast<T>(a.ci);
    const int m1 = wavenum(col, N) - o1;
    const T x1 = static_cast<T>(m1) * il, ec = e1[col];
    cx<T> c[MM + 1];
#pragma unroll
    for (int k = 0; k <= MM; ++k) {
      const c64 ck = sh.coefG[k];
      c[k] = cx<T>{uniform(static_cast<T>(ck.re)), uniform(static_cast<T>(ck.im))};
    }
#pragma unroll 2
    for (int s = 0; s < S::E; ++s) {
      const int pos = jc + s * S::TPL, m2 = wavenum(pos, N) - o2;
      cx<T>& slot = data[G::padded(pos) * S::PITCH + col];
      const T sg = ((col + pos) & 1) ? T(-1) : T(1);
      const T x2 = static_cast<T>(m2) * il;
      const cx<T> w{x1, -x2};
      cx<T> g = c[MM];
#pragma unroll
      for (int k = MM - 1; k >= 0; --k) g = cfma(w, g, c[k]);
      const T r2 = fmar(x1, x1, x2 * x2);
      T ir2;
      if constexpr (sizeof(T) == 8) ir2 = recip_newton(r2);
      else ir2 = recip(r2);
      ir2 = sg * ci * ir2;
      // (where e^{-|xi - a|^2} is zero the polynomial may not be finite)
      const T eg = ec * e2[pos];
      const cx<T> gs{eg > T(0) ? eg * g.re : T(0), eg > T(0) ? eg * g.im : T(0)};
      const cx<T> sv = sg * cf * slot - gs;
      cx<T> r{(sv.re * x1 + sv.im * x2) * ir2, (sv.im * x1 - sv.re * x2) * ir2};
      if (m1 == 0 && m2 == 0) r = cvt<T>((sg * a.ci) * sh.coefG[kMaxM + 1]);
      slot = r;
    }
  }
#pragma unroll
  for (int s = 0; s < S::E; ++s) v[s] = data[G::padded(jc + s * S::TPL) * S::PITCH + col];
  __syncthreads();
  line_fft<T, G, 1, S::PITCH, false>(v, jc, data + col, tw, nullptr);
#pragma unroll
  for (int s = 0; s < S::E; ++s) data[G::padded(jc + s * S::TPL) * S::PITCH + col] = v[s];
  __syncthreads();
#pragma unroll
  for (int s = 0; s < S::E; ++s) v[s] = data[G::padded(row) * S::PITCH + jt + s * S::TPL];
  __syncthreads();
  line_fft<T, G, 1, 1, false>(v, jt, data + row * G::LDS_LINE, tw, nullptr);
}

// v (row layout): F^{-1}R -> alpha s + beta q_k conj(h) with h = F^{-1}R + tail; the sums of |.|^2 and of <s, .>
template <typename T, int N, int MM>
DBAR_D void small_result(const LineArgs& a, int b, cx<T>* v, int row, int jt, SmallShared<T, N>& sh, double alpha,
                         c64 beta, const cx<T>* s_in, double& nrm, double& sdot) {
  using S = SmallGeom<T, N>;
  using G = typename S::G;
  cx<T>* my = reinterpret_cast<cx<T>*>(sh.data) + row * G::LDS_LINE;
  cx<T> d[kMaxM + 1];
#pragma unroll
  for (int n = 0; n <= kMaxM; ++n) d[n] = n <= MM ? cx<T>{uniform(sh.d[n].re), uniform(sh.d[n].im)} : cx<T>{T(0), T(0)};
  cx<T> ey{T(1), T(0)};
  const size_t eo = (size_t)b * a.e_bs;
  if constexpr (sizeof(T) == 8) ey = a.ey[eo + row];
  else ey = a.ey32[eo + row];
  const cx<T>* Q = static_cast<const cx<T>*>(a.Q) + (size_t)b * a.Q_bs + (size_t)row * N;
  const T y = xgrid_t<T, N>(row, a.L);
#pragma unroll
  for (int s = 0; s < S::E; ++s) my[G::padded(jt + s * S::TPL)] = v[s];
  constexpr int GROUP = 4;  // reads of four elements in flight together
#pragma unroll 1
  for (int s0 = 0; s0 < S::E; s0 += GROUP) {
    cx<T> q[GROUP], ex[GROUP], tab[GROUP], si[GROUP];
#pragma unroll
    for (int u = 0; u < GROUP; ++u) {
      const int pos = jt + (s0 + u) * S::TPL;
      q[u] = Q[pos];
      if constexpr (sizeof(T) == 8) ex[u] = a.ex[eo + pos];
      else ex[u] = a.ex32[eo + pos];
      tab[u] = static_cast<const cx<T>*>(a.ttab)[tail_index<N>(row, pos)];
      si[u] = s_in ? s_in[row * N + pos] : cx<T>{T(0), T(0)};
    }
#pragma unroll
    for (int u = 0; u < GROUP; ++u) {
      const int pos = jt + (s0 + u) * S::TPL;
      cx<T>& slot = my[G::padded(pos)];
      const T x = xgrid_t<T, N>(pos, a.L);
      const cx<T> t = tail_tab<T, MM>(x, y, d, tab[u]);
      const cx<T> ph = ex[u] * ey;
      // shifted: h = F^{-1}R + e^{i a.x} tail and q alone; else q_k = q e_k
      const cx<T> h = a.shv ? slot + conj(ph) * t : slot + t;
      const cx<T> w = (a.shv ? q[u] : q[u] * ph) * conj(h);
      cx<T> ot;
      if constexpr (sizeof(T) == 8) ot = beta * w + alpha * si[u];
      else ot = cvt<T>(beta) * w + static_cast<T>(alpha) * si[u];
      slot = ot;
      nrm += rdot(ot, ot);
      sdot += rdot(si[u], ot);
    }
  }
#pragma unroll
  for (int s = 0; s < S::E; ++s) v[s] = my[G::padded(jt + s * S::TPL)];
}

template <typename T, int N, bool ITERATED, int MM>
__global__ void __launch_bounds__((SmallGeom<T, N>::NT), (SmallGeom<T, N>::NW >= 8 ? 2 : 1))
    k_small_cycle(SmallArgs sa) {
  using S = SmallGeom<T, N>;
  constexpr size_t n = (size_t)N * N;
  __shared__ SmallShared<T, N> sh;
  const int b = blockIdx.x;
  if (!sa.act[b]) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Ctl& c = sa.ctl[b];
  cx<T>* V = static_cast<cx<T>*>(sa.V) + (size_t)b * sa.V_bs;
  if (threadIdx.x == 0) {
    sh.sigma[0] = c.sigma[0];
    sh.g[0] = c.g[0];
  }
  for (int t = threadIdx.x; t < kMaxM1 * kMaxM1; t += S::NT) sh.binom[t] = kBinom.v[t / kMaxM1][t % kMaxM1];
  if (threadIdx.x < kMaxM1) sh.invfact[threadIdx.x] = kInvFact[threadIdx.x];
  for (int t = threadIdx.x; t < N; t += S::NT) {
    const double y = xgrid<N>(t, sa.first.L);
    double p = 1.0;
    for (int l = 0; l <= kMaxM + 1; ++l) {
      sh.ypow[t * (kMaxM + 2) + l] = p;
      p *= y;
    }
    const LineArgs* pass[2] = {&sa.first, &sa.second};
    for (int k = 0; k < (ITERATED ? 2 : 1); ++k) {
      const int* o = pass[k]->shv ? pass[k]->shv + 2 * b : nullptr;
      for (int c = 0; c < 2; ++c) {
        const double xi = (wavenum(t, N) - (o ? o[c] : 0)) / sa.first.L;
        sh.e1[k][c][t] = static_cast<T>(exp(-xi * xi));
      }
    }
  }
  double resid = 0.0;
  const double thresh = c.thresh;
  const bool windowed = sa.window > 0 && !sa.act[2 * sa.fs + b];
  bool stopped = false, restart = false;  // first wave: left the cycle, by the restart length
  int steps = 0;
  cx<T> v[S::E];
#pragma unroll
  for (int s = 0; s < S::E; ++s) v[s] = V[(threadIdx.x / S::TPL) * N + threadIdx.x % S::TPL + s * S::TPL];

  for (int j = 0; j < sa.mlim; ++j) {
    const cx<T>* Vj = V + (size_t)j * n;
    double nrm = 0.0, sdot = 0.0;
    const int tid = fresh(threadIdx.x), row = tid / S::TPL, jt = tid % S::TPL;
    small_inverse<T, N, MM, 0>(sa.first, b, v, row, jt, sh, sa.wscale);
    if constexpr (ITERATED) {
      double x0 = 0.0, x1 = 0.0;
      small_result<T, N, MM>(sa.first, b, v, row, jt, sh, 0.0, c64{0.0, -1.0}, nullptr, x0, x1);
      small_inverse<T, N, MM, 1>(sa.second, b, v, row, jt, sh, sa.wscale);
      small_result<T, N, MM>(sa.second, b, v, row, jt, sh, 1.0, c64{0.0, 1.0}, Vj, nrm, sdot);
    } else {
      small_result<T, N, MM>(sa.first, b, v, row, jt, sh, 1.0, c64{0.0, 1.0}, Vj, nrm, sdot);
    }
    // products with v_lo .. v_j and |w|^2: one partial per wave and value
    const int lo = windowed ? (j - sa.window + 1 > 0 ? j - sa.window + 1 : 0) : 0;
    const int nv = j - lo + 1;
    double x;
    if (nv == 2) {  // a windowed step: its three sums side by side
      double p = 0.0;
#pragma unroll
      for (int s = 0; s < S::E; ++s) p += rdot(sh.prev[s * S::NT + tid], v[s]);
      p = wsum(p);
      sdot = wsum(sdot);
      nrm = wsum(nrm);
      if (lane == 0) {
        sh.red[wave] = p;
        sh.red[S::NW + wave] = sdot;
        sh.red[2 * S::NW + wave] = nrm;
      }
    } else {
      sdot = wsum(sdot);
      nrm = wsum(nrm);
      if (lane == 0) {
        sh.red[(nv - 1) * S::NW + wave] = sdot;
        sh.red[nv * S::NW + wave] = nrm;
      }
#pragma unroll 1
      for (int i = 0; i < nv - 1; ++i) {
        const cx<T>* Vi = V + (size_t)(lo + i) * n + row * N;
        double p4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < S::E; ++s) p4[s & 3] += rdot(Vi[jt + s * S::TPL], v[s]);
        x = wsum((p4[0] + p4[1]) + (p4[2] + p4[3]));
        if (lane == 0) sh.red[i * S::NW + wave] = x;
      }
    }
    __syncthreads();
    // first wave: coefficients and, from |w|^2 and the products, the early convergence decision (k_ctl_coef)
    if (wave == 0) {
      const bool in = lane >= lo && lane <= j;
      double h = 0.0, wn2 = 0.0;
      if (in)
        for (int q = 0; q < S::NW; ++q) h += sh.red[(lane - lo) * S::NW + q];
      for (int q = 0; q < S::NW; ++q) wn2 += sh.red[nv * S::NW + q];
      const double sg = in ? sh.sigma[lane] : 0.0, hsum = sg * h;
      if (lane <= j) {
        sh.hsum[lane] = hsum;
        sh.coef[lane] = sg * hsum;
      }
      const double b2 = wn2 - wsum(hsum * hsum);
      bool stop = false;
      if (b2 > 1e-4 * wn2) {
        const double beta = sqrt(b2);
        double mine;
        const double top = small_column(sh, j, mine);
        const double sub = sh.sigma[j] * beta, den = hypot(top, sub);
        const double est = den > 0.0 ? fabs(sub / den * sh.g[j]) : 0.0;
        if (est <= thresh || j + 1 >= sa.m) {
          resid = small_givens(c, sh, j, beta, top, mine);
          stop = stopped = true;
          restart = est > thresh;
          steps = j + 1;
        }
      }
      if (lane == 0) sh.stop = stop;
    }
    __syncthreads();
    if (sh.stop) break;
    // v_{j+1} = w - sum coef_i v_i (FP64), its norm
    {
      c64 w[S::E];
#pragma unroll
      for (int s = 0; s < S::E; ++s) w[s] = cvt<double>(v[s]);
#pragma unroll 1
      for (int i = lo; i < j - 1; ++i) {
        const double cf = sh.coef[i];
        const cx<T>* Vi = V + (size_t)i * n + row * N;
#pragma unroll
        for (int s = 0; s < S::E; ++s) w[s] = w[s] - cf * cvt<double>(Vi[jt + s * S::TPL]);
      }
      const bool two = j - 1 >= lo;
      const double cp = two ? sh.coef[j - 1] : 0.0, cj = sh.coef[j];
      const cx<T>* Vr = Vj + row * N;
#pragma unroll
      for (int s = 0; s < S::E; ++s) {
        const cx<T> vj = Vr[jt + s * S::TPL];
        if (two) w[s] = w[s] - cp * cvt<double>(sh.prev[s * S::NT + tid]);
        w[s] = w[s] - cj * cvt<double>(vj);
        sh.prev[s * S::NT + tid] = vj;
      }
      cx<T>* out = V + (size_t)(j + 1) * n + row * N;
      nrm = 0.0;
#pragma unroll
      for (int s = 0; s < S::E; ++s) {
        v[s] = cvt<T>(w[s]);
        out[jt + s * S::TPL] = v[s];
        nrm += rdot(v[s], v[s]);
      }
    }
    x = wsum(nrm);
    if (lane == 0) sh.red[wave] = x;
    __syncthreads();
    if (wave == 0) {
      double b2 = 0.0;
      for (int q = 0; q < S::NW; ++q) b2 += sh.red[q];
      const double beta = sqrt(b2 > 0.0 ? b2 : 0.0);
      double mine;
      const double top = small_column(sh, j, mine);
      resid = small_givens(c, sh, j, beta, top, mine);
      steps = j + 1;
      stopped = resid <= thresh || j + 1 >= sa.m || beta == 0.0;
      restart = resid > thresh && j + 1 >= sa.m && beta != 0.0;
      if (lane == 0) sh.stop = stopped;
    }
    __syncthreads();
    if (sh.stop) break;
  }
  if (wave == 0) {
    if (lane < steps) {
      c.sigma[lane] = sh.sigma[lane];
      c.g[lane] = sh.g[lane];
      c.cs[lane] = sh.cs[lane];
      c.sn[lane] = sh.sn[lane];
    }
    if (lane == 0) {
      c.resid = resid;
      c.jn = steps;
      c.iters += steps;
      if (stopped) sa.act[b] = 0;
      if (restart) sa.act[sa.fs + b] = 1;
      atomicMax(sa.act + 3 * sa.fs, steps);
    }
  }
}

template <typename T, int N>
void launch_n(const SmallArgs& sa, int B, int method, hipStream_t s) {
  constexpr int NT = SmallGeom<T, N>::NT;
  const bool m11 = sa.first.M == 11;  // the order the loops are unrolled for: the order itself, or the largest
  if (method == 1 && m11) hipLaunchKernelGGL((k_small_cycle<T, N, true, 11>), dim3(B), dim3(NT), 0, s, sa);
  else if (method == 1) hipLaunchKernelGGL((k_small_cycle<T, N, true, kMaxM>), dim3(B), dim3(NT), 0, s, sa);
  else if (m11) hipLaunchKernelGGL((k_small_cycle<T, N, false, 11>), dim3(B), dim3(NT), 0, s, sa);
  else hipLaunchKernelGGL((k_small_cycle<T, N, false, kMaxM>), dim3(B), dim3(NT), 0, s, sa);
}

}  // namespace

// N = 8 has fewer elements than a wave has lanes.  Where |xi|^2 or its reciprocal leaves the normal range, the division's
// Newton steps do not hold.  And on domains so large that the grid holds a potential in one point, the value of h there is a
// sum that cancels exactly in the order of the launches per stage, but only to rounding here, which L multiplies: with
// L = 1e5 such a solve stops at a residual of 4e-14 instead of 1e-16, with 1e12 (mixed) and 1e20 it does not converge.
bool small_cycle_ok(int N, double L) { return (N == 16 || N == 32 || N == 64) && L > 1e-100 && L < 1e3; }

template <typename T>
void launch_small_cycle(const Pipeline& P, Work& w, int method, int window, int mlim, hipStream_t s) {
  const int B = w.B;
  int* act = static_cast<int*>(w.act.p);
  SmallArgs sa;
  sa.first = P.base(B, act, method == 1 ? kShifted : 0u);
  sa.first.tw = sizeof(T) == 8 ? P.tw64 : P.tw32;
  sa.first.Q = sizeof(T) == 8 ? w.Q64.p : w.Q32.p;
  sa.first.Q_bs = w.Q_bs;
  sa.first.ttab = sizeof(T) == 8 ? P.tail64 : P.tail32;
  sa.second = sa.first;
  if (method == 1) {
    sa.second = P.base(B, act, kUnitPhase);
    sa.second.tw = sa.first.tw;
    sa.second.ttab = sa.first.ttab;
    sa.second.Q = sa.first.Q;
    sa.second.Q_bs = sa.first.Q_bs;
  }
  sa.V = w.V.p;
  sa.V_bs = w.n * (w.m + 1);
  sa.ctl = static_cast<Ctl*>(w.ctl.p);
  sa.act = act;
  sa.fs = w.flag_stride;
  sa.m = w.m;
  sa.mlim = mlim;
  sa.window = window;
  const double dx = 2.0 * kPi * P.L / P.N;
  sa.wscale = dx * dx / (2.0 * kPi);
  // (the steps differ by entry and are not known here: v_0 read and, per step, about the window read twice and one written)
  TimerScope ts(kStageCycle + (sizeof(T) == 4), (double)w.n * sizeof(cx<T>), B, act, s);
  switch (P.N) {
    case 16: launch_n<T, 16>(sa, B, method, s); break;
    case 32: launch_n<T, 32>(sa, B, method, s); break;
    default: launch_n<T, 64>(sa, B, method, s); break;
  }
}
template void launch_small_cycle<double>(const Pipeline&, Work&, int, int, int, hipStream_t);
template void launch_small_cycle<float>(const Pipeline&, Work&, int, int, int, hipStream_t);

}  // namespace dbar
