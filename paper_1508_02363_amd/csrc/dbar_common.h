// Common device/host definitions for the D-bar GPU library (gfx950).
//
// Complex numbers are stored interleaved (re, im) in 8- or 16-byte aligned pairs.  All arrays on an N x N grid are
// row-major: x-space arrays a[iy][ix] with x_j = L(-pi + 2 pi j/N); xi-space arrays A[p2][p1] in FFT order, where
// the index p stands for the wave number m = p (p <= N/2) or m = p - N (p > N/2) and xi = m / L (paper Section 4.1,
// equations 'domain' and 'xidomain': the Nyquist wave number is +N/(2L)).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define DBAR_HD __host__ __device__ __forceinline__
#define DBAR_D __device__ __forceinline__

namespace dbar {

constexpr int kMaxM = 15;          // largest Taylor order M supported (the paper uses M = 11, at most about 20)
constexpr int kNMom = kMaxM + 2;   // moments d_0..d_M plus the conj(z) moment
constexpr double kPi = 3.14159265358979323846;

template <typename T>
struct alignas(2 * sizeof(T)) cx {
  T re, im;
};
using c64 = cx<double>;
using c32 = cx<float>;

template <typename T> DBAR_HD cx<T> mk(T a, T b) { return cx<T>{a, b}; }
template <typename T> DBAR_HD cx<T> operator+(cx<T> a, cx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T> DBAR_HD cx<T> operator-(cx<T> a, cx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <typename T> DBAR_HD cx<T> operator-(cx<T> a) { return {-a.re, -a.im}; }
template <typename T> DBAR_HD cx<T> operator*(cx<T> a, cx<T> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename T> DBAR_HD cx<T> operator*(T s, cx<T> a) { return {s * a.re, s * a.im}; }
template <typename T> DBAR_HD cx<T> conj(cx<T> a) { return {a.re, -a.im}; }
template <typename T> DBAR_HD cx<T> mul_i(cx<T> a) { return {-a.im, a.re}; }     // i * a
template <typename T> DBAR_HD cx<T> mul_mi(cx<T> a) { return {a.im, -a.re}; }    // -i * a
template <typename T> DBAR_HD T norm2(cx<T> a) { return a.re * a.re + a.im * a.im; }

DBAR_HD float fmar(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
DBAR_HD double fmar(double a, double b, double c) { return __builtin_fma(a, b, c); }
// a * b + c as four fused multiply-adds (the operators above take six instructions for it: the addition of c cannot
// be contracted into the product's last step)
template <typename T> DBAR_HD cx<T> cfma(cx<T> a, cx<T> b, cx<T> c) {
  return {fmar(a.re, b.re, fmar(-a.im, b.im, c.re)), fmar(a.re, b.im, fmar(a.im, b.re, c.im))};
}
// Re(conj(a) b) as a double, for FP64 accumulation.  FP32 data: the product is formed in FP32 (one fused rounding);
// its error, relative to |a||b| per element and of random sign, is below what the FP32 data carry themselves.
template <typename T> DBAR_HD double rdot(cx<T> a, cx<T> b) {
  if constexpr (sizeof(T) == 4) return static_cast<double>(fmar(a.im, b.im, a.re * b.re));
  else return a.re * b.re + a.im * b.im;
}

template <typename To, typename From> DBAR_HD cx<To> cvt(cx<From> a) {
  return cx<To>{static_cast<To>(a.re), static_cast<To>(a.im)};
}

// ------------------------------------------------------------------------------------------------------------
// Exchanges between the lanes of a wave (all 64 active) without LDS: __shfl_xor is a trip through the LDS crossbar per
// 32-bit word (about a hundred cycles on a reduction's serial chain, and the CU's waves share the crossbar), a DPP move
// or a half-wave swap is one vector instruction.  Same pairs, same sums.  With every wave reduction on them (and the moments
// halved over groups of any size, below): one application at N = 1024 78.8 -> 74.8 us, one solve at N = 128 752 -> 719 us,
// nine iterated ones at N = 512 1.135 -> 1.111 ms, 63 at N = 256 1.737 -> 1.691 ms.
// ------------------------------------------------------------------------------------------------------------
template <int CTRL>
DBAR_D int dpp_word(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}
// a and b's 32-bit words with b's lanes whose bit OFF (16 or 32) is clear and a's whose bit is set changing places:
// a becomes {a's clear, b's clear}, b {a's set, b's set}
template <int OFF>
DBAR_D void swap_words(int& a, int& b) {
  static_assert(OFF == 16 || OFF == 32, "rows of sixteen or half waves");
  if constexpr (OFF == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
  }
}
template <int OFF>
DBAR_D void swap_lanes(float& a, float& b) {
  int x = __builtin_bit_cast(int, a), y = __builtin_bit_cast(int, b);
  swap_words<OFF>(x, y);
  a = __builtin_bit_cast(float, x);
  b = __builtin_bit_cast(float, y);
}
template <int OFF>
DBAR_D void swap_lanes(double& a, double& b) {
  const long long x = __builtin_bit_cast(long long, a), y = __builtin_bit_cast(long long, b);
  int xl = (int)x, xh = (int)(x >> 32), yl = (int)y, yh = (int)(y >> 32);
  swap_words<OFF>(xl, yl);
  swap_words<OFF>(xh, yh);
  a = __builtin_bit_cast(double, (long long)(((unsigned long long)(unsigned)xh << 32) | (unsigned)xl));
  b = __builtin_bit_cast(double, (long long)(((unsigned long long)(unsigned)yh << 32) | (unsigned)yl));
}
// the word of lane ^ OFF, OFF = 1, 2, 4, 8: quad permutations, half-row mirror after a quad mirror, row rotation
template <int OFF>
DBAR_D int xor_word(int x) {
  static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8, "within a row of sixteen lanes");
  if constexpr (OFF == 1) return dpp_word<0xB1>(x);
  else if constexpr (OFF == 2) return dpp_word<0x4E>(x);
  else if constexpr (OFF == 4) return dpp_word<0x141>(dpp_word<0x1B>(x));
  else return dpp_word<0x128>(x);
}
template <int OFF>
DBAR_D float xor_lane(float x) { return __builtin_bit_cast(float, xor_word<OFF>(__builtin_bit_cast(int, x))); }
template <int OFF>
DBAR_D double xor_lane(double x) {
  const long long v = __builtin_bit_cast(long long, x);
  const unsigned lo = xor_word<OFF>((int)v), hi = xor_word<OFF>((int)(v >> 32));
  return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}
// x + the x of lane ^ OFF
template <int OFF, typename T>
DBAR_D T add_xor(T x) {
  if constexpr (OFF >= 16) {
    T y = x;
    swap_lanes<OFF>(x, y);
    return x + y;
  } else {
    return x + xor_lane<OFF>(x);
  }
}
// sum over the wave, in every lane
DBAR_D double wsum(double x) {
  return add_xor<1>(add_xor<2>(add_xor<4>(add_xor<8>(add_xor<16>(add_xor<32>(x))))));
}

// Sums of NV values over the lanes that differ in the bits OFF, OFF / 2, .., LAST: while their number is even each step
// halves them (lanes with the bit clear keep the lower half, the others the upper half, each summed with its partner's
// copy), else it adds in place.  A lane ends with values base .. base + reduce_left() - 1 (base returned) in x[0 ..].
template <int NV, int OFF, int LAST>
constexpr int reduce_left() {
  if constexpr (OFF < LAST) return NV;
  else return reduce_left<(NV % 2 ? NV : NV / 2), OFF / 2, LAST>();
}
// the bits of the steps that added in place: lanes that differ in them alone hold the same sums
template <int NV, int OFF, int LAST>
constexpr int reduce_copies() {
  if constexpr (OFF < LAST) return 0;
  else return (NV % 2 ? OFF : 0) | reduce_copies<(NV % 2 ? NV : NV / 2), OFF / 2, LAST>();
}
template <int NV, int OFF, int LAST, typename T>
DBAR_D int reduce_lanes(T* x, int lane) {
  if constexpr (OFF < LAST) {
    return 0;
  } else if constexpr (NV % 2 == 0) {
    constexpr int H = NV / 2;
    const bool hi = (lane & OFF) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      if constexpr (OFF >= 16) {
        swap_lanes<OFF>(x[i], x[i + H]);
        x[i] = x[i] + x[i + H];
      } else {
        const T keep = hi ? x[i + H] : x[i], send = hi ? x[i] : x[i + H];
        x[i] = keep + xor_lane<OFF>(send);
      }
    }
    return (hi ? H : 0) + reduce_lanes<H, OFF / 2, LAST>(x, lane);
  } else {
#pragma unroll
    for (int i = 0; i < NV; ++i) x[i] = add_xor<OFF>(x[i]);
    return reduce_lanes<NV, OFF / 2, LAST>(x, lane);
  }
}

DBAR_HD int ilog2(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return l;
}

// Wave number index p -> signed wave number m in [-N/2+1, N/2].
DBAR_HD int wavenum(int p, int N) { return p <= N / 2 ? p : p - N; }

}  // namespace dbar
