// Upward and downward transfers of one node by columns (device code; the
// transfer kernels and the spectral zones' fused ones).  A workgroup of 256
// threads per parent node or leaf.
#pragma once

#include "internal.h"

namespace pfmm {
namespace {

constexpr int kColThreads = 256;

template <class W> __device__ inline const W* wsel(Weights w);
template <> __device__ inline const float* wsel<float>(Weights w) { return w.f; }
template <> __device__ inline const double* wsel<double>(Weights w) { return w.d; }

// M2M and L2L, the eight children in one pass per axis.  The child operators
// are T_o = T_ox (x) T_oy (x) T_oz with two 1D matrices T_0, T_1, so along each
// axis the two children of a pair share the pass: M2M contracts x over (ox, kx)
// for the four (oy, oz), then y over (oy, ky) for the two oz, then z over (oz,
// kz) (14 p^4 multiply-adds against 24 p^4 child by child); L2L expands x into
// the two ox, y into four (ox, oy), z into the eight children.
//
// A lane takes whole columns (the values along the contracted axis in
// registers, from memory in the first pass), a wave the outputs whose weights
// it reads as scalars: an LDS value is read once for several outputs and no
// weight is read from LDS.  Reading both factors of every product from LDS was
// the bound, and child by child (p other than 4 and 8) the barriers.  Measured
// before / after: 64 parents in FP64 M2M 33 / 5 us at p = 7, 17 / 4.5 at p = 6, 11 /
// 5.5 at p = 8, L2L 23 / 4.0, 13 / 3.9 and 7.5 / 5.5; 4096 parents of FP32 children, p =
// 8, M2M 207 / 27 us.
// LDS rows are padded to an odd number of values.

// LDS values of m2m_block and l2l_block
template <int P>
constexpr int pair_words() { return 6 * P * P * (P | 1); }

// Masses of parent B from its children; store(i, v) takes parent value i.
template <class TI, class W, int P, class STORE>
__device__ __forceinline__ void m2m_block(const TI* __restrict__ Mc, const W* __restrict__ T, int np, int B,
                                          W* lds, STORE&& store) {
  constexpr int P2 = P * P, P3 = P2 * P, Q = P | 1;
  W* w = lds;               // [oy][oz][ax][ky][kz]
  W* v = lds + 4 * P2 * Q;  // [oz][ax][ay][kz]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int Bx = B / (np * np), By = (B / np) % np, Bz = B % np;
  const int nc = 2 * np;
  for (int c = lane; c < P2; c += 64) {  // (ky, kz) of the wave's (oy, oz)
    W in[2 * P];
#pragma unroll
    for (int ox = 0; ox < 2; ++ox) {
      const size_t child = ((size_t)(2 * Bx + ox) * nc + (2 * By + (wave >> 1))) * nc + (2 * Bz + (wave & 1));
#pragma unroll
      for (int kx = 0; kx < P; ++kx) in[ox * P + kx] = (W)Mc[child * P3 + kx * P2 + c];
    }
#pragma unroll
    for (int ax = 0; ax < P; ++ax) {
      W acc = 0;
#pragma unroll
      for (int k = 0; k < 2 * P; ++k) acc += T[((k / P) * P + ax) * P + k % P] * in[k];
      w[((wave * P + ax) * P + c / P) * Q + c % P] = acc;
    }
  }
  __syncthreads();
  for (int c = lane; c < P2; c += 64) {  // (ax, kz) of oz = wave % 2, every other ay
    const int oz = wave & 1, ax = c / P, kz = c % P;
    W in[2 * P];
#pragma unroll
    for (int k = 0; k < 2 * P; ++k) in[k] = w[((((k / P) * 2 + oz) * P + ax) * P + k % P) * Q + kz];
#pragma unroll
    for (int i = 0; i < (P + 1) / 2; ++i) {
      const int ay = 2 * i + (wave >> 1);
      if (ay >= P) break;
      W acc = 0;
#pragma unroll
      for (int k = 0; k < 2 * P; ++k) acc += T[((k / P) * P + ay) * P + k % P] * in[k];
      v[((oz * P + ax) * P + ay) * Q + kz] = acc;
    }
  }
  __syncthreads();
  for (int c = lane; c < P2; c += 64) {  // (ax, ay), every fourth az
    W in[2 * P];
#pragma unroll
    for (int k = 0; k < 2 * P; ++k) in[k] = v[((k / P) * P2 + c) * Q + k % P];
#pragma unroll
    for (int i = 0; i < (P + 3) / 4; ++i) {
      const int az = 4 * i + wave;
      if (az >= P) break;
      W acc = 0;
#pragma unroll
      for (int k = 0; k < 2 * P; ++k) acc += T[((k / P) * P + az) * P + k % P] * in[k];
      store(c * P + az, acc);
    }
  }
}

// Parent B's local values, load(i), expanded to its children.
template <class TO, class W, int P, class LOAD>
__device__ __forceinline__ void l2l_block(LOAD&& load, TO* __restrict__ Pc, const W* __restrict__ T, int np,
                                          int B, int accumulate, W* lds) {
  constexpr int P2 = P * P, P3 = P2 * P, Q = P | 1;
  W* w = lds;               // [ox][bx][ay][az]
  W* v = lds + 2 * P2 * Q;  // [ox][oy][bx][by][az]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int Bx = B / (np * np), By = (B / np) % np, Bz = B % np;
  const int nc = 2 * np;
  for (int c = lane; c < P2; c += 64) {  // (ay, az) of ox = wave % 2, every other bx
    const int ox = wave & 1;
    W in[P];
#pragma unroll
    for (int a = 0; a < P; ++a) in[a] = load(a * P2 + c);
#pragma unroll
    for (int i = 0; i < (P + 1) / 2; ++i) {
      const int bx = 2 * i + (wave >> 1);
      if (bx >= P) break;
      W acc = 0;
#pragma unroll
      for (int a = 0; a < P; ++a) acc += T[(ox * P + a) * P + bx] * in[a];
      w[((ox * P + bx) * P + c / P) * Q + c % P] = acc;
    }
  }
  __syncthreads();
  for (int c = lane; c < P2; c += 64) {  // (bx, az) of (ox, oy) = wave
    const int bx = c / P, az = c % P;
    W in[P];
#pragma unroll
    for (int a = 0; a < P; ++a) in[a] = w[(((wave >> 1) * P + bx) * P + a) * Q + az];
#pragma unroll
    for (int by = 0; by < P; ++by) {
      W acc = 0;
#pragma unroll
      for (int a = 0; a < P; ++a) acc += T[((wave & 1) * P + a) * P + by] * in[a];
      v[((wave * P + bx) * P + by) * Q + az] = acc;
    }
  }
  __syncthreads();
  for (int c = lane; c < P2; c += 64) {  // (bx, by) of (ox, oy) = wave
    W in[P];
#pragma unroll
    for (int a = 0; a < P; ++a) in[a] = v[(wave * P2 + c) * Q + a];
#pragma unroll
    for (int oz = 0; oz < 2; ++oz) {
      const size_t child = ((size_t)(2 * Bx + (wave >> 1)) * nc + (2 * By + (wave & 1))) * nc + (2 * Bz + oz);
      TO* dst = Pc + child * P3 + c * P;
#pragma unroll
      for (int bz = 0; bz < P; ++bz) {
        W acc = 0;
#pragma unroll
        for (int a = 0; a < P; ++a) acc += T[(oz * P + a) * P + bz] * in[a];
        dst[bz] = accumulate ? (TO)((W)dst[bz] + acc) : (TO)acc;
      }
    }
  }
}

// P2M and L2P of leaves of 4, 8 or 16 cells by columns, as M2M and L2L: a lane
// holds a column of cells or nodes in registers, the weights are scalars.  P2M
// contracts z, y, x (mesh rows in the first pass), L2P expands z, y, x (the last
// pass writes the mesh, its prior values read before the first).  Any
// alignment.  FP32 gridlets of p = 4 and 8 at s = 8 and 16 keep the row kernels of
// updown.hip (k_p2m, k_l2p): L2P is no faster here (256^3, p = 8: 35 us there, 34 here;
// 512^3 247 and 262), and P2M, which is faster (29 and 24, 175 and 159), would sum
// in another order: results would move by their FP32 rounding, which L2P's
// extrapolation amplifies at leaf corners, and be no closer to FP64.  Bound:
// latency of the three passes up to some 10^3 leaves, then the mesh's traffic.
// Measured before (one output a thread, both factors of every product from LDS) /
// after, FP64 gridlets, 512 leaves of s = 16, p = 6: P2M 18 / 8 us, L2P 20 / 6; p = 8,
// 19 / 6 and 23 / 5.5.

template <int S, int P>
constexpr int p2m_col_words() { return (S * S + S * P) * (P | 1); }
template <int S, int P>
constexpr int l2p_col_words() { return P * P * (S + 1) + P * S * S; }

// Masses of leaf b; store(i, v) takes value i.
template <class TR, class W, int S, int P, class STORE>
__device__ __forceinline__ void p2m_block(const TR* __restrict__ rho, const W* __restrict__ A, int N, int b,
                                          W h3, int vec, W* lds, STORE&& store) {
  constexpr int P2 = P * P, Q = P | 1;
  constexpr bool kHalves = S * P <= kColThreads / 2;
  W* t1 = lds;              // [cx][cy][az]
  W* t2 = lds + S * S * Q;  // [cx][ay][az]
  const int nL = N / S;
  const int bx = b / (nL * nL), by = (b / nL) % nL, bz = b % nL;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  {
    // threads of a row set share the az: whole waves (scalar weights) from S = 8 on
    constexpr int G = kColThreads / (S * S);
    const int r = tid % (S * S), g = G == 1 ? 0 : S == 8 ? wave : tid / (S * S);
    const TR* src = rho + ((size_t)(bx * S + r / S) * N + (by * S + r % S)) * N + (size_t)bz * S;
    TR row[S];
    if (vec) {
      constexpr int V = 16 / sizeof(TR);
      typedef TR vec_t __attribute__((ext_vector_type(V)));
#pragma unroll
      for (int q = 0; q < S / V; ++q) {
        const vec_t x = reinterpret_cast<const vec_t*>(src)[q];
#pragma unroll
        for (int i = 0; i < V; ++i) row[V * q + i] = x[i];
      }
    } else {
#pragma unroll
      for (int c = 0; c < S; ++c) row[c] = src[c];
    }
#pragma unroll
    for (int i = 0; i < (P + G - 1) / G; ++i) {
      const int az = G * i + g;
      if (az >= P) break;
      W acc = 0;
#pragma unroll
      for (int c = 0; c < S; ++c) acc += A[az * S + c] * (W)row[c];
      t1[r * Q + az] = acc;
    }
  }
  __syncthreads();
  const int col = kHalves ? tid % (kColThreads / 2) : tid, h = kHalves ? wave >> 1 : 0;
  if (col < S * P) {
    const int cx = col / P, az = col % P;
    W in[S];
#pragma unroll
    for (int c = 0; c < S; ++c) in[c] = t1[(cx * S + c) * Q + az];
    constexpr int step = kHalves ? 2 : 1;
#pragma unroll
    for (int i = 0; i < (P + step - 1) / step; ++i) {
      const int ay = step * i + h;
      if (ay >= P) break;
      W acc = 0;
#pragma unroll
      for (int c = 0; c < S; ++c) acc += A[ay * S + c] * in[c];
      t2[(cx * P + ay) * Q + az] = acc;
    }
  }
  __syncthreads();
  for (int c = lane; c < P2; c += 64) {  // (ay, az), every fourth ax
    W in[S];
#pragma unroll
    for (int x = 0; x < S; ++x) in[x] = t2[(x * P + c / P) * Q + c % P];
#pragma unroll
    for (int i = 0; i < (P + 3) / 4; ++i) {
      const int ax = 4 * i + wave;
      if (ax >= P) break;
      W acc = 0;
#pragma unroll
      for (int x = 0; x < S; ++x) acc += A[ax * S + x] * in[x];
      store(ax * P2 + c, h3 * acc);
    }
  }
}

// Leaf b's local values, load(i), at its cells: phi (+)= scale times them.
template <class TP, class W, int S, int P, class LOAD>
__device__ __forceinline__ void l2p_block(LOAD&& load, TP* __restrict__ phi, const W* __restrict__ Ax,
                                          const W* __restrict__ Ay, const W* __restrict__ Az, W scale, int N,
                                          int b, int accumulate, W* lds) {
  constexpr int P2 = P * P, G = kColThreads / (S * S);
  constexpr int SX = S / G > 0 ? S / G : 1;  // cx per thread of the last pass
  constexpr bool kHalves = S * P <= kColThreads / 2;
  constexpr int step = kHalves ? 2 : 1;
  W* w1 = lds;                  // [ax][ay][cz]
  W* w2 = lds + P2 * (S + 1);   // [ax][cy][cz]
  const int nL = N / S;
  const int bx = b / (nL * nL), by = (b / nL) % nL, bz = b % nL;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int yz = tid % (S * S), x0 = (G == 1 ? 0 : S == 8 ? wave : tid / (S * S)) * SX;
  const bool last = x0 < S;  // S = 4: the first four row sets
  TP* dst = phi + ((size_t)(bx * S + x0) * N + (by * S + yz / S)) * N + (size_t)bz * S + yz % S;
  TP prior[SX];
  if (accumulate && last) {
#pragma unroll
    for (int x = 0; x < SX; ++x) prior[x] = dst[(size_t)x * N * N];
  }
  for (int c = lane; c < P2; c += 64) {  // (ax, ay), every fourth cz
    W in[P];
#pragma unroll
    for (int a = 0; a < P; ++a) in[a] = load(c * P + a);
#pragma unroll
    for (int i = 0; i < S / 4; ++i) {
      const int cz = 4 * i + wave;
      W acc = 0;
#pragma unroll
      for (int a = 0; a < P; ++a) acc += Az[a * S + cz] * in[a];
      w1[c * (S + 1) + cz] = acc;
    }
  }
  __syncthreads();
  const int col = kHalves ? tid % (kColThreads / 2) : tid, h = kHalves ? wave >> 1 : 0;
  if (col < S * P) {
    const int ax = col / S, cz = col % S;
    W in[P];
#pragma unroll
    for (int a = 0; a < P; ++a) in[a] = w1[(ax * P + a) * (S + 1) + cz];
#pragma unroll
    for (int i = 0; i < S / step; ++i) {
      const int cy = step * i + h;
      W acc = 0;
#pragma unroll
      for (int a = 0; a < P; ++a) acc += Ay[a * S + cy] * in[a];
      w2[(ax * S + cy) * S + cz] = acc;
    }
  }
  __syncthreads();
  if (!last) return;
  W in[P];
#pragma unroll
  for (int a = 0; a < P; ++a) in[a] = w2[a * S * S + yz];
#pragma unroll
  for (int x = 0; x < SX; ++x) {
    W acc = 0;
#pragma unroll
    for (int a = 0; a < P; ++a) acc += Ax[a * S + x0 + x] * in[a];
    acc *= scale;
    dst[(size_t)x * N * N] = accumulate ? (TP)((W)prior[x] + acc) : (TP)acc;
  }
}

}  // namespace
}  // namespace pfmm
