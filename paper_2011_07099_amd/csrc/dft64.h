// FP64 DFTs of 1 .. 10 and 16 values in registers, with literal twiddles
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
// cos(2 pi j / n) for the first quarter of n = 20, 28 and 36 (gridlets of 5, 7, 9 and 10)
__device__ constexpr double kQuarter20[6] = {1.0,
                                             0.951056516295153572116,
                                             0.809016994374947424102,
                                             0.587785252292473129169,
                                             0.309016994374947424102,
                                             0.0};
__device__ constexpr double kQuarter28[8] = {1.0,
                                             0.974927912181823607018,
                                             0.900968867902419126236,
                                             0.781831482468029808708,
                                             0.623489801858733530525,
                                             0.433883739117558120475,
                                             0.222520933956314404289,
                                             0.0};
__device__ constexpr double kQuarter36[10] = {1.0,
                                              0.984807753012208059367,
                                              0.93969262078590838405,
                                              0.866025403784438646764,
                                              0.766044443118978035202,
                                              0.642787609686539326323,
                                              0.5,
                                              0.342020143325668733044,
                                              0.173648177666930348852,
                                              0.0};
// what the 53 bits of each leave out, to 106 bits
__device__ constexpr double kLow96[25] = {
    0, 2.7660245814577704e-17, 2.8989898744545369e-17, 1.8546939997825006e-17,
    -2.5463971562308955e-17, -2.3730918112141115e-17, 1.7645047084336677e-17,
    4.8177382976639352e-17, 5.0175421109034514e-17, 1.4073856984728024e-18,
    -5.0286250739071249e-19, 1.201573657194953e-17, -4.8336466567264567e-17,
    2.4563688504510178e-17, -1.647047979025087e-17, 4.7094109405616768e-17,
    0, -1.9433863591039061e-17, -1.0050772696461588e-17,
    -6.0167485066851732e-18, 2.2872495004955609e-17, -7.9910790684617313e-18,
    -9.6076660239015238e-18, 5.1366338547231789e-18, 0};
__device__ constexpr double kLow20[6] = {
    0, 4.0934500900087295e-17, -2.7160576018412531e-17, -7.9347508381900201e-18,
    -2.7160576018412531e-17, 0};
__device__ constexpr double kLow28[8] = {
    0, -1.2323837650624249e-17, -1.9762646853069492e-17, 5.0743203625828678e-18,
    4.7160999205408961e-17, 7.4071890789466767e-20, 1.1412494827220627e-17, 0};
__device__ constexpr double kLow36[10] = {
    0, 3.9051088757992981e-17, -4.3850932840020416e-17, 5.0175421109034514e-17,
    2.1750711742081045e-17, -3.6596079007909491e-17, 0,
    2.0136016534644645e-17, -1.0090493350843633e-17, 0};
template <int N>
__device__ __forceinline__ double cosdq(const double (&q)[N / 4 + 1], int j) {  // cos(2 pi j / N)
  j %= N;
  if (j < 0) j += N;
  if (j <= N / 4) return q[j];
  if (j <= N / 2) return -q[N / 2 - j];
  if (j <= 3 * N / 4) return -q[j - N / 2];
  return q[N - j];
}
// (cos, sin) of 2 pi j / M, M a divisor of 96, 20, 28 or 36
template <int N, int M>
__device__ __forceinline__ double2 twdq(const double (&q)[N / 4 + 1], int j) {
  return make_double2(cosdq<N>(q, j * (N / M)), cosdq<N>(q, j * (N / M) - N / 4));
}
template <int M>
__device__ __forceinline__ double2 twd(int j) {
  static_assert(96 % M == 0 || 20 % M == 0 || 28 % M == 0 || 36 % M == 0, "no literal twiddles");
  if constexpr (96 % M == 0) return twdq<96, M>(kQuarterD, j);
  else if constexpr (20 % M == 0) return twdq<20, M>(kQuarter20, j);
  else if constexpr (28 % M == 0) return twdq<28, M>(kQuarter28, j);
  else return twdq<36, M>(kQuarter36, j);
}
template <int M>
__device__ __forceinline__ double2 twd_low(int j) {  // what twd's 53 bits leave out
  if constexpr (96 % M == 0) return twdq<96, M>(kLow96, j);
  else if constexpr (20 % M == 0) return twdq<20, M>(kLow20, j);
  else if constexpr (28 % M == 0) return twdq<28, M>(kLow28, j);
  else return twdq<36, M>(kLow36, j);
}

__device__ __forceinline__ double2 dadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 dsub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// a exp(-2 pi i j / P) (forward) or a exp(+2 pi i j / P) (INV)
template <int P, bool INV>
__device__ __forceinline__ double2 dtwiddle(double2 a, int j) {
  const double2 w = twd<P>(j);
  const double y = INV ? w.y : -w.y;  // explicit: every kernel rounds the same
  return make_double2(fma(a.x, w.x, -(a.y * y)), fma(a.y, w.x, a.x * y));
}

// i a
__device__ __forceinline__ double2 dturn(double2 a) { return make_double2(-a.y, a.x); }

// Complex numbers of twice the precision (unevaluated sums of two doubles, by
// Dekker's and Knuth's error-free sums and products), for the same DFTs.
struct wide {
  double h, l;
};
struct wide2 {
  wide x, y;
};
__device__ __forceinline__ wide wnorm(double s, double e) {  // |s| >= |e|
#pragma clang fp contract(off)
  const double h = s + e;
  return {h, e - (h - s)};
}
__device__ __forceinline__ wide wneg(wide a) { return {-a.h, -a.l}; }
__device__ __forceinline__ wide wadd(wide a, wide b) {
#pragma clang fp contract(off)
  const double s = a.h + b.h, t = s - a.h;
  return wnorm(s, ((a.h - (s - t)) + (b.h - t)) + (a.l + b.l));
}
__device__ __forceinline__ wide wmul(wide a, wide b) {
#pragma clang fp contract(off)
  const double m = a.h * b.h;
  return wnorm(m, fma(a.h, b.l, fma(a.l, b.h, fma(a.h, b.h, -m))));
}
__device__ __forceinline__ wide2 dadd(wide2 a, wide2 b) { return {wadd(a.x, b.x), wadd(a.y, b.y)}; }
__device__ __forceinline__ wide2 dsub(wide2 a, wide2 b) {
  return {wadd(a.x, wneg(b.x)), wadd(a.y, wneg(b.y))};
}
__device__ __forceinline__ wide2 dturn(wide2 a) { return {wneg(a.y), a.x}; }
template <int P, bool INV>
__device__ __forceinline__ wide2 dtwiddle(wide2 a, int j) {
  const double2 h = twd<P>(j), l = twd_low<P>(j);
  const wide c = {h.x, l.x}, s = INV ? wide{h.y, l.y} : wide{-h.y, -l.y};
  return {wadd(wmul(a.x, c), wneg(wmul(a.y, s))), wadd(wmul(a.y, c), wmul(a.x, s))};
}

template <bool INV, class T>
__device__ __forceinline__ void ddft4(T& a0, T& a1, T& a2, T& a3) {
  const T b0 = dadd(a0, a2), b1 = dsub(a0, a2), b2 = dadd(a1, a3), b3 = dsub(a1, a3);
  const T ib3 = dturn(b3);
  a0 = dadd(b0, b2);
  a2 = dsub(b0, b2);
  a1 = INV ? dadd(b1, ib3) : dsub(b1, ib3);
  a3 = INV ? dsub(b1, ib3) : dadd(b1, ib3);
}

// In-place DFT of P values: P = 4, 8 or 16 (4 Q) by the split n = Q n1 + n2,
// m = m1 + 4 m2; P = 6, 10 by even and odd n; P = 9 by threes; 3, 5, 7 directly.
template <int P, bool INV, class T>
__device__ __forceinline__ void ddft(T (&v)[P]) {
  if constexpr (P == 1) {
    return;
  } else if constexpr (P % 4 != 0 && P % 2 == 0) {
    T e[P / 2], o[P / 2];
#pragma unroll
    for (int n = 0; n < P / 2; ++n) {
      e[n] = v[2 * n];
      o[n] = v[2 * n + 1];
    }
    ddft<P / 2, INV>(e);
    ddft<P / 2, INV>(o);
#pragma unroll
    for (int m = 0; m < P / 2; ++m) {
      const T t = m ? dtwiddle<P, INV>(o[m], m) : o[m];
      v[m] = dadd(e[m], t);
      v[m + P / 2] = dsub(e[m], t);
    }
  } else if constexpr (P == 9) {  // n = 3 n1 + n2, m = m1 + 3 m2
    T w[3][3];
#pragma unroll
    for (int n2 = 0; n2 < 3; ++n2) {
#pragma unroll
      for (int n1 = 0; n1 < 3; ++n1) w[n2][n1] = v[3 * n1 + n2];
      ddft<3, INV>(w[n2]);
    }
#pragma unroll
    for (int m1 = 0; m1 < 3; ++m1) {
      T u[3];
#pragma unroll
      for (int n2 = 0; n2 < 3; ++n2) u[n2] = n2 * m1 ? dtwiddle<9, INV>(w[n2][m1], n2 * m1) : w[n2][m1];
      ddft<3, INV>(u);
#pragma unroll
      for (int m2 = 0; m2 < 3; ++m2) v[m1 + 3 * m2] = u[m2];
    }
  } else if constexpr (P % 4 != 0) {
    T u[P];
#pragma unroll
    for (int n = 0; n < P; ++n) u[n] = v[n];
#pragma unroll
    for (int m = 0; m < P; ++m) {
      T acc = u[0];
#pragma unroll
      for (int n = 1; n < P; ++n) acc = dadd(acc, m ? dtwiddle<P, INV>(u[n], n * m) : u[n]);
      v[m] = acc;
    }
  } else {
    constexpr int Q = P / 4;
    T w[Q][4];
  #pragma unroll
    for (int n2 = 0; n2 < Q; ++n2) {
      w[n2][0] = v[n2];
      w[n2][1] = v[Q + n2];
      w[n2][2] = v[2 * Q + n2];
      w[n2][3] = v[3 * Q + n2];
      ddft4<INV>(w[n2][0], w[n2][1], w[n2][2], w[n2][3]);
  #pragma unroll
      for (int m1 = 1; m1 < 4; ++m1)
        if (n2) w[n2][m1] = dtwiddle<P, INV>(w[n2][m1], n2 * m1);
    }
  #pragma unroll
    for (int m1 = 0; m1 < 4; ++m1) {
      if constexpr (Q == 1) {
        v[m1] = w[0][m1];
      } else if constexpr (Q == 2) {
        v[m1] = dadd(w[0][m1], w[1][m1]);
        v[m1 + 4] = dsub(w[0][m1], w[1][m1]);
      } else {
        ddft4<INV>(w[0][m1], w[1][m1], w[2][m1], w[3][m1]);
        v[m1] = w[0][m1];
        v[m1 + 4] = w[1][m1];
        v[m1 + 8] = w[2][m1];
        v[m1 + 12] = w[3][m1];
      }
    }
  }
}

}  // namespace
}  // namespace pfmm
