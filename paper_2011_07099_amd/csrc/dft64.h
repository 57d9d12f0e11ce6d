// FP64 DFTs of 4, 6, 8 and 16 values in registers, with literal twiddles
// (device code; shared by the spectral zones and the FP64 near zone).
#pragma once

#include <hip/hip_runtime.h>

namespace pfmm {
namespace {

// cos(2 pi j / 96) for j = 0 .. 24 (96 = lcm of the grid sizes 8, 12, 16, 32)
__device__ constexpr double kQuarterD[25] = {
    1.0,                    0.997858923238603506738, 0.991444861373810411145,
    0.980785280403230449126, 0.96592582628906828675,  0.946930129495105664256,
    0.923879532511286756128, 0.896872741532688303894, 0.866025403784438646764,
    0.831469612302545237079, 0.79335334029123516458,  0.751839807478977396408,
    0.707106781186547524401, 0.659345815100068868425, 0.608761429008720639416,
    0.555570233019602224743, 0.5,                     0.442288690219001281995,
    0.382683432365089771728, 0.321439465303161580701, 0.258819045102520762349,
    0.195090322016128267848, 0.130526192220051591548, 0.0654031292301430668153,
    0.0};
__device__ __forceinline__ double cosd96(int j) {
  j %= 96;
  if (j < 0) j += 96;
  if (j <= 24) return kQuarterD[j];
  if (j <= 48) return -kQuarterD[48 - j];
  if (j <= 72) return -kQuarterD[j - 48];
  return kQuarterD[96 - j];
}

// (cos, sin) of 2 pi j / M, M | 96
template <int M>
__device__ __forceinline__ double2 twd(int j) {
  constexpr int r = 96 / M;
  return make_double2(cosd96(j * r), cosd96(j * r - 24));
}

__device__ __forceinline__ double2 dadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 dsub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// a exp(-2 pi i j / P) (forward) or a exp(+2 pi i j / P) (INV)
template <int P, bool INV>
__device__ __forceinline__ double2 dtwiddle(double2 a, int j) {
  const double2 w = twd<P>(j);
  return INV ? make_double2(a.x * w.x - a.y * w.y, a.y * w.x + a.x * w.y)
             : make_double2(a.x * w.x + a.y * w.y, a.y * w.x - a.x * w.y);
}

template <bool INV>
__device__ __forceinline__ void ddft4(double2& a0, double2& a1, double2& a2, double2& a3) {
  const double2 b0 = dadd(a0, a2), b1 = dsub(a0, a2), b2 = dadd(a1, a3), b3 = dsub(a1, a3);
  const double2 ib3 = make_double2(-b3.y, b3.x);
  a0 = dadd(b0, b2);
  a2 = dsub(b0, b2);
  a1 = INV ? dadd(b1, ib3) : dsub(b1, ib3);
  a3 = INV ? dsub(b1, ib3) : dadd(b1, ib3);
}

// In-place DFT of P values: P = 4Q (Q = 1, 2, 4) by the split n = Q n1 + n2,
// m = m1 + 4 m2; P = 6 directly.
template <int P, bool INV>
__device__ __forceinline__ void ddft(double2 (&v)[P]) {
  if constexpr (P == 6) {
    double2 u[6];
#pragma unroll
    for (int n = 0; n < 6; ++n) u[n] = v[n];
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      double2 acc = u[0];
#pragma unroll
      for (int n = 1; n < 6; ++n) acc = dadd(acc, dtwiddle<6, INV>(u[n], n * m));
      v[m] = acc;
    }
    return;
  }
  constexpr int Q = P / 4;
  double2 T[Q][4];
#pragma unroll
  for (int n2 = 0; n2 < Q; ++n2) {
    T[n2][0] = v[n2];
    T[n2][1] = v[Q + n2];
    T[n2][2] = v[2 * Q + n2];
    T[n2][3] = v[3 * Q + n2];
    ddft4<INV>(T[n2][0], T[n2][1], T[n2][2], T[n2][3]);
#pragma unroll
    for (int m1 = 1; m1 < 4; ++m1)
      if (n2) T[n2][m1] = dtwiddle<P, INV>(T[n2][m1], n2 * m1);
  }
#pragma unroll
  for (int m1 = 0; m1 < 4; ++m1) {
    if constexpr (Q == 1) {
      v[m1] = T[0][m1];
    } else if constexpr (Q == 2) {
      v[m1] = dadd(T[0][m1], T[1][m1]);
      v[m1 + 4] = dsub(T[0][m1], T[1][m1]);
    } else {
      ddft4<INV>(T[0][m1], T[1][m1], T[2][m1], T[3][m1]);
      v[m1] = T[0][m1];
      v[m1 + 4] = T[1][m1];
      v[m1 + 8] = T[2][m1];
      v[m1 + 12] = T[3][m1];
    }
  }
}

}  // namespace
}  // namespace pfmm
