// Device helpers of the GMRES control steps, shared by the control kernels and the whole-cycle kernel of small grids.
#pragma once

#include "dbar_solver.h"

namespace dbar {

// 1/n!, n <= kMaxM + 1
static __constant__ double kInvFact[kMaxM + 2] = {
    1.0, 1.0, 5.0e-1, 1.6666666666666666e-1, 4.1666666666666664e-2, 8.3333333333333332e-3,
    1.3888888888888889e-3, 1.9841269841269841e-4, 2.4801587301587302e-5, 2.7557319223985893e-6,
    2.7557319223985888e-7, 2.5052108385441720e-8, 2.0876756987868100e-9, 1.6059043836821613e-10,
    1.1470745597729725e-11, 7.6471637318198164e-13, 4.7794773323873853e-14};

// *flag as one thread reads it, in every thread of the block: for a flag that another block of the launch may clear
// meanwhile, where waves that read it for themselves could part, some past the block's barriers and some not.  A barrier
// behind a load the launch begins with anyway.
DBAR_D int block_flag(const int* flag) {
  __shared__ int f;
  if (threadIdx.x == 0) f = *flag;
  __syncthreads();
  return f;
}

// lane l's x in every lane (l uniform: a register read, not a trip through LDS as __shfl is)
DBAR_D double bcast(double x, int l) {
  const long long v = __builtin_bit_cast(long long, x);
  const unsigned lo = __builtin_amdgcn_readlane((int)v, l), hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// c_n from d_n: (-i/2)^n d_n / n! (equation fourreeg4 with Gchoice; (-i/2)^n = (-i)^n 2^-n exactly)
DBAR_D c64 taylor_power(int n, c64 d) {  // (-i/2)^n d
  const double s = ldexp(1.0, -n);
  const c64 p = s * d;
  return (n & 3) == 0 ? p : (n & 3) == 1 ? mul_mi(p) : (n & 3) == 2 ? -p : mul_i(p);
}
DBAR_D c64 taylor_coef(int n, c64 d) { return kInvFact[n] * taylor_power(n, d); }

// sum of p[0 .. nblk) over one wave (every lane gets it), in an order fixed by nblk.  Eight independent partial sums
// per lane: the loads of a chunk are in flight together.
DBAR_D double wave_reduce(const double* __restrict__ p, int nblk) {
  double a[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  int i = threadIdx.x & 63;
  for (; i + 7 * 64 < nblk; i += 8 * 64) {
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] += p[i + u * 64];
  }
#pragma unroll
  for (int u = 0; u < 7; ++u)
    if (i + u * 64 < nblk) a[u] += p[i + u * 64];
  return wsum(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])));
}

// One Hessenberg column in a wave's registers: lane i holds sigma_i, hsum_i and rotation i, and the rotations run
// through all of them with register reads (a single thread that walks the record in memory waits for each term).
struct HessLane {
  double cs, sn, raw;  // raw: the column's entry i before the rotations, sigma_j hsum_i
  int first;           // the first entry that can be nonzero after them (rotation i mixes entries i and i + 1)
};
DBAR_D HessLane hess_lane(double cs, double sn, double sigma_j, int j, double hsum) {
  const int lane = threadIdx.x & 63;
  HessLane h;
  h.cs = cs;
  h.sn = sn;
  h.raw = lane <= j ? sigma_j * hsum : 0.0;
  const unsigned long long nz = __ballot(h.raw != 0.0);
  const int f = nz ? __builtin_ctzll(nz) : j;
  h.first = f > 0 ? f - 1 : 0;
  return h;
}
DBAR_D HessLane hess_lane(const Ctl& c, int j, double hsum) {
  const int lane = threadIdx.x & 63;
  return hess_lane(lane < j ? c.cs[lane] : 1.0, lane < j ? c.sn[lane] : 0.0, c.sigma[j], j, hsum);
}
// entry j of the rotated column (every lane); mine: entry `lane` for lane < j
DBAR_D double hess_rotate(const HessLane& h, int j, double& mine) {
  const int lane = threadIdx.x & 63;
  double top = bcast(h.raw, h.first);
  mine = 0.0;
  for (int i = h.first; i < j; ++i) {
    const double c = bcast(h.cs, i), s = bcast(h.sn, i), next = bcast(h.raw, i + 1);
    if (lane == i) mine = c * top + s * next;
    top = -s * top + c * next;
  }
  return top;
}

// Column j of the Hessenberg matrix from hsum and beta = ||v_{j+1}|| (unnormalised basis: column j is sigma_j times the
// products of A v_j), the previous Givens rotations applied, the new rotation, g and the residual estimate |g_{j+1}|.
// One whole wave (top, mine: hess_rotate's); returns the estimate.
DBAR_D double givens_commit(Ctl& c, int j, double beta, double top, double mine) {
  const int lane = threadIdx.x & 63;
  double* col = c.H + (size_t)j * (kMaxRestart + 1);
  const double sub = c.sigma[j] * beta, gj = c.g[j];
  const double den = hypot(top, sub);
  const double cs = den > 0.0 ? top / den : 1.0, sn = den > 0.0 ? sub / den : 0.0;
  const double resid = fabs(-sn * gj);
  if (lane < j) col[lane] = mine;
  if (lane == 0) {
    col[j] = den;
    col[j + 1] = 0.0;
    c.sigma[j + 1] = beta > 0.0 ? 1.0 / beta : 0.0;
    c.cs[j] = cs;
    c.sn[j] = sn;
    c.g[j + 1] = -sn * gj;
    c.g[j] = cs * gj;
    c.resid = resid;
    c.jn = j + 1;
    c.iters += 1;
  }
  return resid;
}

// Gram-Schmidt pass `pass` of step j: h_i = <v_i, w> from the partials, coef_i = sigma_i^2 h_i (the basis is kept
// unnormalised, v_i / ||v_i|| = sigma_i v_i), hsum_i accumulates sigma_i h_i over the passes.  One block per entry.
// early (one pass, value j + 1 of the partials = ||w||^2): the step's convergence is decided here, before the update
// that forms v_{j+1} runs.  With one classical pass v_{j+1} = w - sum_i hsum_i q_i (q_i = sigma_i v_i orthonormal), so
// ||v_{j+1}||^2 = ||w||^2 - sum_i hsum_i^2; where that difference keeps at least 1e-4 of ||w||^2 (the FP64 sums of
// products then fix beta to about 1e-3 relative or better), the rotation it implies gives the residual estimate, and
// an entry that meets its threshold (or the restart length) takes its last Givens step with this beta and leaves the
// cycle: the update, transform and moments of a v_{j+1} no step would use are not run for it.  Otherwise the step
// waits for the exact norm from the update, as without `early`.
// The partials cover the vectors lo..j; an entry whose own window starts later (full[b] == 0 with skip > 0: the launch
// covers the whole basis for entries that orthogonalise fully) takes the vectors lo + skip..j only.
DBAR_D void ctl_coef_entry(int b, Ctl* ctl, const double* part, int nval, const TileSpan& span, int* act, int fs, int j,
                           int pass, int early, int m, int lo, int skip, const int* full) {
  __shared__ double red[kMaxRestart + 2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nblk = span.count(b);
  for (int v = wave; v < nval; v += blockDim.x / 64) {
    const double x = wave_reduce(part + ((size_t)b * nval + v) * span.stride, nblk);
    if (lane == 0) red[v] = x;
  }
  __syncthreads();
  if (wave != 0) return;
  Ctl& c = ctl[b];
  const int lob = lo + ((full && !full[b]) ? skip : 0);
  const bool in = lane >= lob && lane <= j;  // outside the window (one pass): zero
  const double sg = in ? c.sigma[lane] : 0.0, h = in ? red[lane - lo] : 0.0;
  const double hsum = in ? (pass ? c.hsum[lane] : 0.0) + sg * h : 0.0;
  if (lane <= j) {
    c.coef[lane] = sg * sg * h;
    c.hsum[lane] = hsum;
  }
  if (early) {
    const double wn2 = red[j - lo + 1], b2 = wn2 - wsum(hsum * hsum);
    if (b2 > 1e-4 * wn2) {
      const double beta = sqrt(b2);
      double mine;
      const HessLane hl = hess_lane(c, j, hsum);
      const double top = hess_rotate(hl, j, mine);
      // the residual estimate with this beta, without touching the record
      const double sub = c.sigma[j] * beta, den = hypot(top, sub);
      const double resid = den > 0.0 ? fabs(sub / den * c.g[j]) : 0.0;
      if (resid <= c.thresh || j + 1 >= m) {
        givens_commit(c, j, beta, top, mine);
        if (lane == 0) {
          act[b] = 0;
          if (resid > c.thresh) act[fs + b] = 1;  // stopped by the restart length
        }
      }
    }
  }
}


}  // namespace dbar
