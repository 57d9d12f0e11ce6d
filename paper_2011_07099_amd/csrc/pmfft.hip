// The exact periodic convolution of Eq. 4,
//   phi_i = h^3 sum_j G((x_i - x_j) wrapped) rho_j,
// by the convolution theorem: FP64 transforms of the N^3 mesh (N a power of
// two, 8 .. 1024), multiplied by the transform of G sampled at every mesh
// separation.  Exact up to FP64 rounding; results rounded once to FP32.
//
// Five passes over the half spectrum [N][N][N/2 + 1]: real rows along z, lines
// along y, lines along x forward, times G's transform, and back in one pass,
// lines along y, rows along z.  A workgroup transforms its lines in LDS.  The
// forward passes along y and x take their lines in natural order to
// bit-reversed order (decimation in frequency), the inverse ones back, and G's
// transform is made by the same passes, so nothing is ever reordered.
//
// Each pass reads and writes the spectrum once: at 64^3 launches and latency
// bound it, from 256^3 on HBM.  36 us at 64^3, 78 us at 128^3, 0.46 ms at 256^3;
// the direct sum it replaces (2 N^6 flops) took 14.6 ms at 64^3.
#include "internal.h"

#include <algorithm>

namespace pfmm {
namespace {

constexpr int kThreads = 256;
constexpr int kLdsValues = 2048;  // values of the lines a workgroup transforms

inline unsigned nblk(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }

// tw[k] = exp(-2 pi i k / N), k < N / 2
__device__ __forceinline__ void twiddles(int N, double2* tw) {
  for (int k = threadIdx.x; k < N / 2; k += kThreads) sincospi(-2.0 * k / N, &tw[k].y, &tw[k].x);
}

// `lines` (a power of two) transforms of N = 2^lg values in LDS, value n of
// line c at buf[n sn + c sc]; ends with a barrier.  Two radix-2 stages a pass.
// Forward: natural to bit-reversed order.  Inverse (unnormalised): back.
template <bool INV, bool ROWS>
__device__ void fft_lines(double2* buf, const double2* tw, int lg, int lglines, int sn, int sc) {
  const int N = 1 << lg, lines = 1 << lglines;
  // butterfly b of `per` a line -> (index along the line, line); rows: the
  // index runs fastest over the lanes, else the line
  auto split = [&](int b, int lgper, int& j, int& c) {
    j = ROWS ? b & ((1 << lgper) - 1) : b >> lglines;
    c = ROWS ? b >> lgper : b & (lines - 1);
  };
  auto two = [&](int lgh) {  // one stage of half-length 2^lgh
    const int h = 1 << lgh;
    for (int b = threadIdx.x; b < (N / 2) * lines; b += kThreads) {
      int j, c;
      split(b, lg - 1, j, c);
      const int m = j & (h - 1), i = ((j >> lgh) << (lgh + 1)) + m;
      double2* p = buf + i * sn + c * sc;
      const double2 w = tw[m << (lg - 1 - lgh)], a = p[0], d = p[h * sn];
      if (INV) {
        const double2 t = cmul(d, cconj(w));
        p[0] = cadd(a, t);
        p[h * sn] = csub(a, t);
      } else {
        p[0] = cadd(a, d);
        p[h * sn] = cmul(csub(a, d), w);
      }
    }
    __syncthreads();
  };
  auto four = [&](int lgq) {  // the stages of half-lengths 2^(lgq + 1) and 2^lgq
    const int q = 1 << lgq;
    for (int b = threadIdx.x; b < (N / 4) * lines; b += kThreads) {
      int j, c;
      split(b, lg - 2, j, c);
      const int m = j & (q - 1), i = ((j >> lgq) << (lgq + 2)) + m, s = lg - 2 - lgq;
      double2* p = buf + i * sn + c * sc;
      const double2 x0 = p[0], x1 = p[q * sn], x2 = p[2 * q * sn], x3 = p[3 * q * sn];
      const double2 w0 = tw[m << s], w1 = tw[(m + q) << s], v = tw[m << (s + 1)];
      if (INV) {
        const double2 t1 = cmul(x1, cconj(v)), t3 = cmul(x3, cconj(v));
        const double2 y0 = cadd(x0, t1), y1 = csub(x0, t1);
        const double2 y2 = cmul(cadd(x2, t3), cconj(w0)), y3 = cmul(csub(x2, t3), cconj(w1));
        p[0] = cadd(y0, y2);
        p[2 * q * sn] = csub(y0, y2);
        p[q * sn] = cadd(y1, y3);
        p[3 * q * sn] = csub(y1, y3);
      } else {
        const double2 y0 = cadd(x0, x2), y2 = cmul(csub(x0, x2), w0);
        const double2 y1 = cadd(x1, x3), y3 = cmul(csub(x1, x3), w1);
        p[0] = cadd(y0, y1);
        p[q * sn] = cmul(csub(y0, y1), v);
        p[2 * q * sn] = cadd(y2, y3);
        p[3 * q * sn] = cmul(csub(y2, y3), v);
      }
    }
    __syncthreads();
  };
  if (INV) {
    int l = 0;
    for (; l + 2 <= lg; l += 2) four(l);
    if (l < lg) two(l);
  } else {
    int l = lg;
    if (l & 1) two(--l);
    for (; l > 0; l -= 2) four(l - 2);
  }
}

__device__ __forceinline__ int bitrev(int k, int lg) { return (int)(__brev((unsigned)k) >> (32 - lg)); }

// Real rows along z to half spectra, two rows (y, y + 1) as one complex line;
// LDS: 2^lgpairs lines of N + 1 values, then the twiddles.
template <class T>
__global__ void __launch_bounds__(kThreads) k_pm_rows(const T* __restrict__ in, int lg, int lgpairs,
                                                      double2* __restrict__ out) {
  extern __shared__ __align__(16) double2 sm[];
  const int N = 1 << lg, H = N / 2 + 1, pairs = 1 << lgpairs;
  double2* tw = sm + pairs * (N + 1);
  twiddles(N, tw);
  const int64_t pair0 = (int64_t)blockIdx.x * pairs;
  for (int i = threadIdx.x; i < pairs * N; i += kThreads) {
    const int c = i >> lg, n = i & (N - 1);
    const T* row = in + (pair0 + c) * 2 * N + n;
    sm[c * (N + 1) + n] = make_double2((double)row[0], (double)row[N]);
  }
  __syncthreads();
  fft_lines<false, true>(sm, tw, lg, lgpairs, 1, N + 1);
  for (int i = threadIdx.x; i < pairs * H; i += kThreads) {
    const int c = i / H, k = i % H;
    const double2 a = sm[c * (N + 1) + bitrev(k, lg)], b = cconj(sm[c * (N + 1) + bitrev((N - k) & (N - 1), lg)]);
    double2* o = out + (pair0 + c) * 2 * H + k;
    o[0] = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y + b.y));
    o[H] = make_double2(0.5 * (a.y - b.y), -0.5 * (a.x - b.x));
  }
}

// Half spectra along z back to two real rows each (the imaginary parts of the
// zero and Nyquist values, rounding, are left out).
__global__ void __launch_bounds__(kThreads) k_pm_rows_inv(const double2* __restrict__ in, int lg, int lgpairs,
                                                          float* __restrict__ out) {
  extern __shared__ __align__(16) double2 sm[];
  const int N = 1 << lg, H = N / 2 + 1, pairs = 1 << lgpairs;
  double2* tw = sm + pairs * (N + 1);
  twiddles(N, tw);
  const int64_t pair0 = (int64_t)blockIdx.x * pairs;
  for (int i = threadIdx.x; i < pairs * H; i += kThreads) {
    const int c = i / H, k = i % H;
    const double2* p = in + (pair0 + c) * 2 * H + k;
    double2 a = p[0], b = p[H];
    if (k == 0 || k == N / 2) a.y = b.y = 0.0;
    sm[c * (N + 1) + bitrev(k, lg)] = make_double2(a.x - b.y, a.y + b.x);
    if (k > 0 && k < N / 2) sm[c * (N + 1) + bitrev(N - k, lg)] = make_double2(a.x + b.y, b.x - a.y);
  }
  __syncthreads();
  fft_lines<true, true>(sm, tw, lg, lgpairs, 1, N + 1);
  for (int i = threadIdx.x; i < pairs * N; i += kThreads) {
    const int c = i >> lg, n = i & (N - 1);
    const double2 v = sm[c * (N + 1) + n];
    float* row = out + (pair0 + c) * 2 * N + n;
    row[0] = (float)v.x;
    row[N] = (float)v.y;
  }
}

// Lines along y (axis 1) or x (axis 0) of the half spectrum, in place, for one
// plane and 2^lgcols neighbouring kz.  MODE 0: forward; 1: inverse; 2: forward,
// times g, inverse.
template <int MODE>
__global__ void __launch_bounds__(kThreads) k_pm_lines(double2* __restrict__ a, int lg, int lgcols, int axis,
                                                       const double2* __restrict__ g) {
  extern __shared__ __align__(16) double2 sm[];
  const int N = 1 << lg, H = N / 2 + 1, cols = 1 << lgcols;
  double2* tw = sm + cols * N;
  twiddles(N, tw);
  const int nblock = (H + cols - 1) >> lgcols;
  const int plane = blockIdx.x / nblock, k0 = (blockIdx.x % nblock) << lgcols;
  const int64_t base = (axis ? (int64_t)plane * N : (int64_t)plane) * H + k0;
  const int64_t step = axis ? H : (int64_t)N * H;
  for (int i = threadIdx.x; i < cols * N; i += kThreads) {
    const int c = i & (cols - 1), n = i >> lgcols;
    sm[i] = k0 + c < H ? a[base + n * step + c] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  if (MODE != 1) fft_lines<false, false>(sm, tw, lg, lgcols, cols, 1);
  if (MODE == 2) {
    for (int i = threadIdx.x; i < cols * N; i += kThreads) {
      const int c = i & (cols - 1), n = i >> lgcols;
      if (k0 + c < H) sm[i] = cmul(sm[i], g[base + n * step + c]);
    }
    __syncthreads();
  }
  if (MODE != 0) fft_lines<true, false>(sm, tw, lg, lgcols, cols, 1);
  for (int i = threadIdx.x; i < cols * N; i += kThreads) {
    const int c = i & (cols - 1), n = i >> lgcols;
    if (k0 + c < H) a[base + n * step + c] = sm[i];
  }
}

// log2 of the lines a workgroup takes: at most 16 (256-byte runs along kz), at
// most what there is, kLdsValues values in all.
int lines_of(int lg, int most) {
  int l = 0;
  while (l < most && (2 << (l + lg)) <= kLdsValues) ++l;
  return l;
}

template <class T>
hipError_t rows(const T* in, int lg, double2* out, hipStream_t st) {
  const int N = 1 << lg, lp = lines_of(lg, 2 * lg - 1);
  const size_t lds = ((size_t)(N + 1) * (1 << lp) + N / 2) * sizeof(double2);
  k_pm_rows<T><<<(unsigned)(((int64_t)N * N / 2) >> lp), kThreads, lds, st>>>(in, lg, lp, out);
  return hipGetLastError();
}

template <int MODE>
hipError_t lines(double2* a, int lg, int axis, const double2* g, hipStream_t st) {
  const int N = 1 << lg, H = N / 2 + 1, lc = lines_of(lg, 4);
  const size_t lds = ((size_t)N * (1 << lc) + N / 2) * sizeof(double2);
  const unsigned blocks = (unsigned)N * (unsigned)((H + (1 << lc) - 1) >> lc);
  k_pm_lines<MODE><<<blocks, kThreads, lds, st>>>(a, lg, lc, axis, g);
  return hipGetLastError();
}

// N = 2^lg, 8 .. 1024 (the lines and twiddles then fit in 41 KiB of LDS)
int log2_of(int N) {
  int lg = 3;
  while (lg < 10 && (1 << lg) < N) ++lg;
  return (1 << lg) == N ? lg : -1;
}

}  // namespace

size_t pm_values(int N) { return (size_t)N * N * (N / 2 + 1); }

hipError_t pm_kernel(const double* tab, int C, int N, double2* work, double2* ghat, hipStream_t st) {
  const int lg = log2_of(N);
  if (lg < 0 || 2 * C < N) return hipErrorInvalidValue;
  const double n6 = (double)N * N * N * (double)N * N * N;  // h^3 and the unnormalised transforms
  double* mesh = reinterpret_cast<double*>(work);
  hipError_t e = gstar_mesh_values(tab, C, N, 1.0 / n6, mesh, st);
  if (e == hipSuccess) e = rows(mesh, lg, ghat, st);
  if (e == hipSuccess) e = lines<0>(ghat, lg, 1, nullptr, st);
  if (e == hipSuccess) e = lines<0>(ghat, lg, 0, nullptr, st);
  return e;
}

hipError_t pm_convolve(const float* rho, const double2* ghat, double2* work, int N, float* phi, hipStream_t st) {
  const int lg = log2_of(N);
  if (lg < 0) return hipErrorInvalidValue;
  hipError_t e = rows(rho, lg, work, st);
  if (e == hipSuccess) e = lines<0>(work, lg, 1, nullptr, st);
  if (e == hipSuccess) e = lines<2>(work, lg, 0, ghat, st);
  if (e == hipSuccess) e = lines<1>(work, lg, 1, nullptr, st);
  if (e != hipSuccess) return e;
  const int lp = lines_of(lg, 2 * lg - 1);
  const size_t lds = ((size_t)(N + 1) * (1 << lp) + N / 2) * sizeof(double2);
  k_pm_rows_inv<<<(unsigned)(((int64_t)N * N / 2) >> lp), kThreads, lds, st>>>(work, lg, lp, phi);
  return hipGetLastError();
}

}  // namespace pfmm
