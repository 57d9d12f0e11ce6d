// Upward and downward passes of the FMM on the uniform tree (Sec. 2):
//   P2M  leaf cells -> leaf gridlet (effective masses with the same Cartesian
//        moments 0 <= n_i < p; the 1D weights are the Lagrange basis of the
//        gridlet nodes evaluated at the cell centres),
//   M2M  Eq. 5, child gridlets -> parent gridlet,
//   L2L  Eq. 7, parent local field -> child gridlets (the transposed operator,
//        i.e. Lagrange interpolation),
//   L2P  leaf gridlet -> cells (transpose of P2M); with derivative weights on
//        one axis, the gradient of the leaf's local expansion (accelerations
//        from the expansion, Sec. 3),
//   FD4  a = -grad(phi) by periodic 4th-order central differences (Sec. 3).
// Every operator is a tensor product of 1D operators and is applied as three
// successive 1D contractions on a block staged in LDS.  These stages move a
// few bytes per cell and are bound by memory traffic, not arithmetic.
//
// Gridlet buffers of a level are FP32 or FP64 (coarse levels can be kept in
// FP64: the interpolation of Eq. 7 extrapolates past the parent's outermost
// gridlet nodes, so rounding noise of a parent's field is amplified in its
// children); each kernel computes in the wider of its operand types.
#include "columns.h"
#include "internal.h"

namespace pfmm {
namespace {

constexpr int kThreads = 256;

// S, P: leaf width and gridlet size fixed at compile time (0: the arguments),
// so that the index arithmetic folds and the contraction loops unroll.
template <class TO, class W, int S = 0, int P = 0, class TR = float>
__global__ __launch_bounds__(kThreads) void k_p2m(const TR* __restrict__ rho,
                                                   TO* __restrict__ M, Weights Aw, int N, int s_,
                                                   int p_, W h3) {
  const int s = S ? S : s_, p = P ? P : p_;
  // LDS rows of the weights and of the cell block padded by one word, so
  // that lanes reading different rows at one column hit different banks
  const int sp = s + 1;
  // compile-time rows of FP32 cells, one per thread: each thread contracts
  // its own row along z from registers, and the cell block never goes
  // through LDS (a third of the LDS, so more leaves per CU)
  constexpr bool kRowRegs = S % 4 == 0 && S > 0 && P > 0 && S * S <= kThreads &&
                            sizeof(TR) == 4;
  extern __shared__ __align__(8) unsigned char smraw[];
  W* sm = reinterpret_cast<W*>(smraw);
  W* sA = sm;               // [p][s + 1]
  W* sr = sA + p * sp;      // [s][s][s + 1] (not with rows in registers)
  W* t1 = kRowRegs ? sr : sr + s * s * sp;  // [cx][cy][az]
  W* t2 = t1 + s * s * p;   // [cx][ay][az]
  const W* A = wsel<W>(Aw);
  const int nL = N / s;
  const int b = (int)xcd_leaf(blockIdx.x, (int64_t)nL * nL * nL);
  const int bx = b / (nL * nL), by = (b / nL) % nL, bz = b % nL;
  const int tid = threadIdx.x;
  if constexpr (kRowRegs) {
    float4 rowv[S / 4];
    if (tid < S * S) {
      const int cx = tid / S, cy = tid % S;
      const float4* src = reinterpret_cast<const float4*>(
          rho + ((size_t)(bx * S + cx) * N + (by * S + cy)) * N + (size_t)bz * S);
#pragma unroll
      for (int q = 0; q < S / 4; ++q) rowv[q] = src[q];
    }
    for (int i = tid; i < P * S; i += kThreads) sA[(i / S) * sp + i % S] = A[i];
    __syncthreads();
    if (tid < S * S) {
#pragma unroll
      for (int az = 0; az < P; ++az) {
        const W* w = sA + az * sp;
        W acc = 0;
#pragma unroll
        for (int q = 0; q < S / 4; ++q)
          acc += w[4 * q] * (W)rowv[q].x + w[4 * q + 1] * (W)rowv[q].y +
                 w[4 * q + 2] * (W)rowv[q].z + w[4 * q + 3] * (W)rowv[q].w;
        t1[tid * P + az] = acc;
      }
    }
    __syncthreads();
  } else {
    for (int i = tid; i < p * s; i += kThreads) sA[(i / s) * sp + i % s] = A[i];
    for (int i = tid; i < s * s * s; i += kThreads) {
      const int cx = i / (s * s), cy = (i / s) % s, cz = i % s;
      sr[(cx * s + cy) * sp + cz] = (W)rho[((size_t)(bx * s + cx) * N + (by * s + cy)) * N + (bz * s + cz)];
    }
    __syncthreads();
    for (int i = tid; i < s * s * p; i += kThreads) {
      const int cxy = i / p, az = i % p;
      W acc = 0;
      for (int cz = 0; cz < s; ++cz) acc += sA[az * sp + cz] * sr[cxy * sp + cz];
      t1[i] = acc;
    }
    __syncthreads();
  }
  for (int i = tid; i < s * p * p; i += kThreads) {
    const int cx = i / (p * p), ay = (i / p) % p, az = i % p;
    W acc = 0;
    for (int cy = 0; cy < s; ++cy) acc += sA[ay * sp + cy] * t1[(cx * s + cy) * p + az];
    t2[i] = acc;
  }
  __syncthreads();
  const int p3 = p * p * p;
  for (int i = tid; i < p3; i += kThreads) {
    const int ax = i / (p * p), ayz = i % (p * p);
    W acc = 0;
    for (int cx = 0; cx < s; ++cx) acc += sA[ax * sp + cx] * t2[cx * p * p + ayz];
    M[(size_t)b * p3 + i] = (TO)(h3 * acc);
  }
}

// out[b s + c] (+)= scale sum_a Wx[ax][cx] Wy[ay][cy] Wz[az][cz] P[b][a]: L2P
// with Wx = Wy = Wz = A and scale 1, or one component of the gradient of the
// leaf's local expansion with the derivative weights on that axis
template <class TI, class W, int S = 0, int PP = 0, class TP = float>
__global__ __launch_bounds__(kThreads) void k_l2p(const TI* __restrict__ P,
                                                   TP* __restrict__ phi, Weights Wxw,
                                                   Weights Wyw, Weights Wzw, W scale, int N,
                                                   int s_, int p_, int accumulate) {
  const int s = S ? S : s_, p = PP ? PP : p_;
  extern __shared__ __align__(8) unsigned char smraw[];
  W* sm = reinterpret_cast<W*>(smraw);
  const int p3 = p * p * p;
  W* sAx = sm;             // [p][s] per axis
  W* sAy = sAx + p * s;
  W* sAz = sAy + p * s;
  W* sp = sAz + p * s;     // [ax][ay][az]
  W* w1 = sp + p3;         // [ax][ay][cz]
  W* w2 = w1 + p * p * s;  // [ax][cy][cz]
  const W* Ax = wsel<W>(Wxw);
  const W* Ay = wsel<W>(Wyw);
  const W* Az = wsel<W>(Wzw);
  const int nL = N / s;
  const int b = (int)xcd_leaf(blockIdx.x, (int64_t)nL * nL * nL);
  const int bx = b / (nL * nL), by = (b / nL) % nL, bz = b % nL;
  const int tid = threadIdx.x;
  // with rows of float4 and accumulation, the mesh values this thread will
  // update are read first, so their latency overlaps the two LDS passes
  constexpr int kRows = (S % 4 == 0 && S > 0 && sizeof(TP) == 4)
                            ? (S * S * (S / 4) + kThreads - 1) / kThreads : 1;
  float4 prior[kRows];
  auto row_ptr = [&](int i) {
    const int cx = i / (s * (s / 4)), cy = (i / (s / 4)) % s, cz0 = 4 * (i % (s / 4));
    return reinterpret_cast<float4*>(phi + ((size_t)(bx * s + cx) * N + (by * s + cy)) * N +
                                     (bz * s + cz0));
  };
  if constexpr (S % 4 == 0 && S > 0 && sizeof(TP) == 4) {
    if (accumulate) {
#pragma unroll
      for (int k = 0; k < kRows; ++k) {
        const int i = tid + k * kThreads;
        if (i < s * s * (s / 4)) prior[k] = *row_ptr(i);
      }
    }
  }
  for (int i = tid; i < p * s; i += kThreads) {
    sAx[i] = Ax[i];
    sAy[i] = Ay[i];
    sAz[i] = Az[i];
  }
  for (int i = tid; i < p3; i += kThreads) sp[i] = (W)P[(size_t)b * p3 + i];
  __syncthreads();
  for (int i = tid; i < p * p * s; i += kThreads) {
    const int xy = i / s, cz = i % s;
    W v = 0;
    for (int k = 0; k < p; ++k) v += sAz[k * s + cz] * sp[xy * p + k];
    w1[i] = v;
  }
  __syncthreads();
  for (int i = tid; i < p * s * s; i += kThreads) {
    const int ax = i / (s * s), cy = (i / s) % s, cz = i % s;
    W v = 0;
    for (int k = 0; k < p; ++k) v += sAy[k * s + cy] * w1[(ax * p + k) * s + cz];
    w2[i] = v;
  }
  __syncthreads();
  if constexpr (S % 4 == 0 && S > 0 && sizeof(TP) == 4) {
    // four consecutive cells of a row per thread, read and written as float4
    // (16-byte aligned: the launcher checks the mesh pointer)
#pragma unroll
    for (int kr = 0; kr < kRows; ++kr) {
      const int i = tid + kr * kThreads;
      if (i >= s * s * (s / 4)) break;
      const int cx = i / (s * (s / 4)), cy = (i / (s / 4)) % s, cz0 = 4 * (i % (s / 4));
      W v[4] = {0, 0, 0, 0};
      for (int k = 0; k < p; ++k) {
        const W a = sAx[k * s + cx];
        const W* w = w2 + k * s * s + cy * s + cz0;
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] += a * w[c];
      }
      float4 r = make_float4((float)(v[0] * scale), (float)(v[1] * scale), (float)(v[2] * scale),
                             (float)(v[3] * scale));
      if (accumulate) {
        const float4 q = prior[kr];
        r = make_float4((float)((W)q.x + v[0] * scale), (float)((W)q.y + v[1] * scale),
                        (float)((W)q.z + v[2] * scale), (float)((W)q.w + v[3] * scale));
      }
      *row_ptr(i) = r;
    }
  } else {
    for (int i = tid; i < s * s * s; i += kThreads) {
      const int cx = i / (s * s), cyz = i % (s * s);
      W v = 0;
      for (int k = 0; k < p; ++k) v += sAx[k * s + cx] * w2[k * s * s + cyz];
      v *= scale;
      const int cy = cyz / s, cz = cyz % s;
      TP* o = phi + ((size_t)(bx * s + cx) * N + (by * s + cy)) * N + (bz * s + cz);
      *o = accumulate ? (TP)((W)*o + v) : (TP)v;
    }
  }
}

template <class TI, class TO, class W, int P>
__global__ __launch_bounds__(kThreads) void k_m2m(const TI* __restrict__ Mc, TO* __restrict__ Mp,
                                                   Weights Tw, int np) {
  __shared__ W lds[pair_words<P>()];
  TO* dst = Mp + (size_t)blockIdx.x * (P * P * P);
  m2m_block<TI, W, P>(Mc, wsel<W>(Tw), np, blockIdx.x, lds, [&](int i, W v) { dst[i] = (TO)v; });
}

template <class TI, class TO, class W, int P>
__global__ __launch_bounds__(kThreads) void k_l2l(const TI* __restrict__ Pp, TO* __restrict__ Pc,
                                                   Weights Tw, int np, int accumulate) {
  __shared__ W lds[pair_words<P>()];
  const TI* src = Pp + (size_t)blockIdx.x * (P * P * P);
  l2l_block<TO, W, P>([&](int i) { return (W)src[i]; }, Pc, wsel<W>(Tw), np, blockIdx.x, accumulate, lds);
}

template <class TR, class TO, class W, int S, int P>
__global__ __launch_bounds__(kThreads) void k_p2m_cols(const TR* __restrict__ rho, TO* __restrict__ M,
                                                        Weights Aw, int N, W h3, int vec) {
  __shared__ W lds[p2m_col_words<S, P>()];
  const int nL = N / S, b = (int)xcd_leaf(blockIdx.x, (int64_t)nL * nL * nL);
  TO* dst = M + (size_t)b * (P * P * P);
  p2m_block<TR, W, S, P>(rho, wsel<W>(Aw), N, b, h3, vec, lds, [&](int i, W v) { dst[i] = (TO)v; });
}

template <class TI, class TP, class W, int S, int P>
__global__ __launch_bounds__(kThreads) void k_l2p_cols(const TI* __restrict__ Pl, TP* __restrict__ phi,
                                                        Weights Wxw, Weights Wyw, Weights Wzw, W scale,
                                                        int N, int accumulate) {
  __shared__ W lds[l2p_col_words<S, P>()];
  const int nL = N / S, b = (int)xcd_leaf(blockIdx.x, (int64_t)nL * nL * nL);
  const TI* src = Pl + (size_t)b * (P * P * P);
  l2p_block<TP, W, S, P>([&](int i) { return (W)src[i]; }, phi, wsel<W>(Wxw), wsel<W>(Wyw), wsel<W>(Wzw),
                         scale, N, b, accumulate, lds);
}

// V consecutive cells along z per thread, their rows read and written as
// vectors (V = 1: any alignment).  Bound: 16 bytes a cell from and to memory in
// FP32; 128^3 14 us with one cell per thread, 9
// by vectors.
template <class T, int V>
__global__ __launch_bounds__(kThreads) void k_fd4(const T* __restrict__ phi,
                                                   T* __restrict__ acc, int N) {
  typedef T vec_t __attribute__((ext_vector_type(V)));
  const size_t n3 = (size_t)N * N * N;
  const size_t i = ((size_t)blockIdx.x * kThreads + threadIdx.x) * V;
  if (i >= n3) return;
  const int z = (int)(i % N), y = (int)((i / N) % N), x = (int)(i / ((size_t)N * N));
  const int mk = N - 1;
  const T inv12h = (T)N / (T)12;
  auto row = [&](int xx, int yy, int zz, T* v) {  // V cells from zz on
    const T* p = phi + ((size_t)(xx & mk) * N + (yy & mk)) * N + (zz & mk);
    if constexpr (V > 1) {
      const vec_t q = *reinterpret_cast<const vec_t*>(p);
#pragma unroll
      for (int c = 0; c < V; ++c) v[c] = q[c];
    } else {
      v[0] = *p;
    }
  };
  T xp2[V], xp1[V], xm1[V], xm2[V], yp2[V], yp1[V], ym1[V], ym2[V];
  row(x + 2, y, z, xp2);
  row(x + 1, y, z, xp1);
  row(x - 1, y, z, xm1);
  row(x - 2, y, z, xm2);
  row(x, y + 2, z, yp2);
  row(x, y + 1, z, yp1);
  row(x, y - 1, z, ym1);
  row(x, y - 2, z, ym2);
  constexpr int K = V > 1 ? 1 : 2;  // vectors on either side that hold the two next cells
  T w[(2 * K + 1) * V];             // cells z - K V ... of the row
#pragma unroll
  for (int k = -K; k <= K; ++k) row(x, y, z + k * V, w + (k + K) * V);
  T g[3][V];
#pragma unroll
  for (int c = 0; c < V; ++c) {
    const T* o = w + K * V + c;
    const T gx = -xp2[c] + (T)8 * xp1[c] - (T)8 * xm1[c] + xm2[c];
    const T gy = -yp2[c] + (T)8 * yp1[c] - (T)8 * ym1[c] + ym2[c];
    const T gz = -o[2] + (T)8 * o[1] - (T)8 * o[-1] + o[-2];
    g[0][c] = -gx * inv12h;
    g[1][c] = -gy * inv12h;
    g[2][c] = -gz * inv12h;
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if constexpr (V > 1) {
      vec_t q;
#pragma unroll
      for (int c = 0; c < V; ++c) q[c] = g[d][c];
      *reinterpret_cast<vec_t*>(acc + d * n3 + i) = q;
    } else {
      acc[d * n3 + i] = g[d][0];
    }
  }
}

__global__ void k_d2f(const double* __restrict__ s, float* __restrict__ d, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) d[i] = (float)s[i];
}

}  // namespace

// LDS words of P2M: the padded weights and cell block, and the two partial
// contractions; without the cell block for the instances that keep the
// rows in registers.
inline size_t p2m_words(int s, int p) {
  return (size_t)(p * (s + 1) + s * s * (s + 1) + s * s * p + s * p * p);
}
inline size_t p2m_words_rows(int s, int p) {
  return (size_t)(p * (s + 1) + s * s * p + s * p * p);
}

namespace {
// P2M, L2P by columns where the leaf has 4, 8 or 16 cells, else the general form
template <class TR, class TO, class W>
hipError_t p2m_any(const TR* rho, TO* M, Weights A, int N, int s, int p, W h3, hipStream_t st) {
  const int nL = N / s;
  const dim3 g(nL * nL * nL), b(kThreads);
  if (s != 4 && s != 8 && s != 16) {
    hipLaunchKernelGGL((k_p2m<TO, W, 0, 0, TR>), g, b, p2m_words(s, p) * sizeof(W), st, rho, M, A, N, s, p, h3);
    return hipGetLastError();
  }
  const int vec = ((uintptr_t)rho & 15) == 0;
  return with_p<1, 10>(p, [&](auto P) {
    constexpr int p_ = decltype(P)::value;
    if (s == 16)
      hipLaunchKernelGGL((k_p2m_cols<TR, TO, W, 16, p_>), g, b, 0, st, rho, M, A, N, h3, vec);
    else if (s == 8)
      hipLaunchKernelGGL((k_p2m_cols<TR, TO, W, 8, p_>), g, b, 0, st, rho, M, A, N, h3, vec);
    else
      hipLaunchKernelGGL((k_p2m_cols<TR, TO, W, 4, p_>), g, b, 0, st, rho, M, A, N, h3, vec);
    return hipGetLastError();
  });
}

template <class TI, class TP, class W>
hipError_t l2p_any(const TI* P, TP* out, Weights Wx, Weights Wy, Weights Wz, W scale, int N, int s, int p,
                   hipStream_t st, int accumulate) {
  const int nL = N / s;
  const dim3 g(nL * nL * nL), b(kThreads);
  if (s != 4 && s != 8 && s != 16) {
    const size_t words = (size_t)(3 * p * s + p * p * p + p * p * s + p * s * s);
    hipLaunchKernelGGL((k_l2p<TI, W, 0, 0, TP>), g, b, words * sizeof(W), st, P, out, Wx, Wy, Wz, scale, N, s,
                       p, accumulate);
    return hipGetLastError();
  }
  return with_p<1, 10>(p, [&](auto Pc) {
    constexpr int p_ = decltype(Pc)::value;
    if (s == 16)
      hipLaunchKernelGGL((k_l2p_cols<TI, TP, W, 16, p_>), g, b, 0, st, P, out, Wx, Wy, Wz, scale, N, accumulate);
    else if (s == 8)
      hipLaunchKernelGGL((k_l2p_cols<TI, TP, W, 8, p_>), g, b, 0, st, P, out, Wx, Wy, Wz, scale, N, accumulate);
    else
      hipLaunchKernelGGL((k_l2p_cols<TI, TP, W, 4, p_>), g, b, 0, st, P, out, Wx, Wy, Wz, scale, N, accumulate);
    return hipGetLastError();
  });
}
}  // namespace

hipError_t launch_p2m(const float* rho, void* M, int m64, Weights A, int N, int s, int p,
                      double h3, hipStream_t st) {
  if (m64) return p2m_any(rho, (double*)M, A, N, s, p, h3, st);
  const float hf = (float)h3;
  // FP32 gridlets of p = 4, 8: rows of cells as float4
  if ((s != 8 && s != 16) || (p != 4 && p != 8) || ((uintptr_t)rho & 15))
    return p2m_any(rho, (float*)M, A, N, s, p, hf, st);
  const int nL = N / s;
  const dim3 g(nL * nL * nL), b(kThreads);
  const size_t sh = p2m_words_rows(s, p) * sizeof(float);
  if (s == 16 && p == 8)
    hipLaunchKernelGGL((k_p2m<float, float, 16, 8>), g, b, sh, st, rho, (float*)M, A, N, s, p, hf);
  else if (s == 8 && p == 8)
    hipLaunchKernelGGL((k_p2m<float, float, 8, 8>), g, b, sh, st, rho, (float*)M, A, N, s, p, hf);
  else if (s == 16)
    hipLaunchKernelGGL((k_p2m<float, float, 16, 4>), g, b, sh, st, rho, (float*)M, A, N, s, p, hf);
  else
    hipLaunchKernelGGL((k_p2m<float, float, 8, 4>), g, b, sh, st, rho, (float*)M, A, N, s, p, hf);
  return hipGetLastError();
}

hipError_t launch_m2m(const void* Mc, int c64, void* Mp, int p64, Weights T, int np, int p,
                      hipStream_t st) {
  if (c64 && !p64) return hipErrorInvalidValue;  // a finer level is never wider than its parent
  const dim3 g(np * np * np), b(kThreads);
  return with_p<1, 10>(p, [&](auto P) {
    constexpr int p_ = decltype(P)::value;
    if (!p64)
      hipLaunchKernelGGL((k_m2m<float, float, float, p_>), g, b, 0, st, (const float*)Mc, (float*)Mp, T, np);
    else if (!c64)
      hipLaunchKernelGGL((k_m2m<float, double, double, p_>), g, b, 0, st, (const float*)Mc, (double*)Mp, T, np);
    else
      hipLaunchKernelGGL((k_m2m<double, double, double, p_>), g, b, 0, st, (const double*)Mc, (double*)Mp, T,
                         np);
    return hipGetLastError();
  });
}

hipError_t launch_l2l(const void* Pp, int p64, void* Pc, int c64, Weights T, int np, int p,
                      hipStream_t st, int accumulate) {
  if (c64 && !p64) return hipErrorInvalidValue;
  const dim3 g(np * np * np), b(kThreads);
  return with_p<1, 10>(p, [&](auto P) {
    constexpr int p_ = decltype(P)::value;
    if (!p64)
      hipLaunchKernelGGL((k_l2l<float, float, float, p_>), g, b, 0, st, (const float*)Pp, (float*)Pc, T, np,
                         accumulate);
    else if (!c64)
      hipLaunchKernelGGL((k_l2l<double, float, double, p_>), g, b, 0, st, (const double*)Pp, (float*)Pc, T, np,
                         accumulate);
    else
      hipLaunchKernelGGL((k_l2l<double, double, double, p_>), g, b, 0, st, (const double*)Pp, (double*)Pc, T,
                         np, accumulate);
    return hipGetLastError();
  });
}

namespace {
hipError_t l2p_axes(const void* P, int p64, float* out, Weights Wx, Weights Wy, Weights Wz,
                    double scale, int N, int s, int p, hipStream_t st, int accumulate) {
  if (p64) return l2p_any((const double*)P, out, Wx, Wy, Wz, scale, N, s, p, st, accumulate);
  const float sc = (float)scale;
  const float* Pf = (const float*)P;
  // FP32 gridlets of p = 4, 8: rows of cells as float4
  if ((s != 8 && s != 16) || (p != 4 && p != 8) || ((uintptr_t)out & 15))
    return l2p_any(Pf, out, Wx, Wy, Wz, sc, N, s, p, st, accumulate);
  const int nL = N / s;
  const dim3 g(nL * nL * nL), b(kThreads);
  const size_t sh = (size_t)(3 * p * s + p * p * p + p * p * s + p * s * s) * sizeof(float);
  if (s == 16 && p == 8)
    hipLaunchKernelGGL((k_l2p<float, float, 16, 8>), g, b, sh, st, Pf, out, Wx, Wy, Wz, sc, N, s, p, accumulate);
  else if (s == 8 && p == 8)
    hipLaunchKernelGGL((k_l2p<float, float, 8, 8>), g, b, sh, st, Pf, out, Wx, Wy, Wz, sc, N, s, p, accumulate);
  else if (s == 16)
    hipLaunchKernelGGL((k_l2p<float, float, 16, 4>), g, b, sh, st, Pf, out, Wx, Wy, Wz, sc, N, s, p, accumulate);
  else
    hipLaunchKernelGGL((k_l2p<float, float, 8, 4>), g, b, sh, st, Pf, out, Wx, Wy, Wz, sc, N, s, p, accumulate);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_l2p(const void* P, int p64, float* phi, Weights A, int N, int s, int p,
                      hipStream_t st, int accumulate) {
  return l2p_axes(P, p64, phi, A, A, A, 1.0, N, s, p, st, accumulate);
}

hipError_t launch_l2p_grad(const void* P, int p64, float* acc, Weights A, Weights Ad,
                           double scale, int N, int s, int p, hipStream_t st) {
  const size_t n3 = (size_t)N * N * N;
  for (int c = 0; c < 3; ++c) {
    const hipError_t e = l2p_axes(P, p64, acc + c * n3, c == 0 ? Ad : A, c == 1 ? Ad : A,
                                  c == 2 ? Ad : A, scale, N, s, p, st, 1);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

namespace {
template <class T>
hipError_t fd4_any(const T* phi, T* acc, int N, hipStream_t st) {
  constexpr int V = 16 / sizeof(T);  // N is a multiple of 8
  const size_t n3 = (size_t)N * N * N;
  if ((((uintptr_t)phi | (uintptr_t)acc) & 15) == 0)
    hipLaunchKernelGGL((k_fd4<T, V>), dim3((unsigned)((n3 / V + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                       st, phi, acc, N);
  else
    hipLaunchKernelGGL((k_fd4<T, 1>), dim3((unsigned)((n3 + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                       phi, acc, N);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_fd4(const float* phi, float* acc, int N, hipStream_t st) { return fd4_any(phi, acc, N, st); }

hipError_t launch_fd4_f64(const double* phi, double* acc, int N, hipStream_t st) {
  return fd4_any(phi, acc, N, st);
}

hipError_t launch_p2m_f64in(const double* rho, void* M, Weights A, int N, int s, int p, double h3,
                            hipStream_t st) {
  return p2m_any(rho, (double*)M, A, N, s, p, h3, st);
}

hipError_t launch_l2p_f64out(const void* P, double* phi, Weights A, int N, int s, int p,
                             hipStream_t st, int accumulate) {
  return l2p_any((const double*)P, phi, A, A, A, 1.0, N, s, p, st, accumulate);
}

hipError_t launch_l2p_grad_f64out(const void* P, double* acc, Weights A, Weights Ad, double scale,
                                  int N, int s, int p, hipStream_t st) {
  const size_t n3 = (size_t)N * N * N;
  for (int c = 0; c < 3; ++c) {
    const hipError_t e = l2p_any((const double*)P, acc + c * n3, c == 0 ? Ad : A, c == 1 ? Ad : A,
                                 c == 2 ? Ad : A, scale, N, s, p, st, 1);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_cast_d2f(const double* src, float* dst, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_d2f, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, dst, n);
  return hipGetLastError();
}

}  // namespace pfmm
