// Device helpers of the GMRES control steps, shared by the control kernels and the whole-cycle kernel of small grids.
#pragma once

#include "dbar_solver.h"

namespace dbar {

static __constant__ double kInvFactC[kMaxM + 2] = {
    1.0, 1.0, 5.0e-1, 1.6666666666666666e-1, 4.1666666666666664e-2, 8.3333333333333332e-3,
    1.3888888888888889e-3, 1.9841269841269841e-4, 2.4801587301587302e-5, 2.7557319223985893e-6,
    2.7557319223985888e-7, 2.5052108385441720e-8, 2.0876756987868100e-9, 1.6059043836821613e-10,
    1.1470745597729725e-11, 7.6471637318198164e-13, 4.7794773323873853e-14};

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
DBAR_D c64 taylor_coef(int n, c64 d) { return kInvFactC[n] * taylor_power(n, d); }

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

}  // namespace dbar
