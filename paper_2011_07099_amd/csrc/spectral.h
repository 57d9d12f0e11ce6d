// The spectral zones' state and the transforms of one node (device code),
// shared by the zone kernels and by those fused with the tree's transfers.
#pragma once

#include "dft64.h"
#include "internal.h"

#include <vector>

namespace pfmm {

struct M2LSpectral {
  int L = 0, p = 0;
  int64_t F = 0;                 // (2p)^2 (p + 1) frequencies per node
  std::vector<double2*> spec;    // per level: [F][nodes]
  double2* out = nullptr;        // [F][nodes] of the level being summed
  std::vector<double2*> khatT;   // per level: [F][kKT] kernel values, offsets of [-3, 3]^3 innermost
  float2* khatT32 = nullptr;     // the leaf level's khatT in FP32 (the FP32 16^3 stencil)
  int f32 = 0;                   // khatT32 follows khatT (kept from the spectral option on)
  void* mem = nullptr;           // the one allocation that holds the arrays above
};

namespace {

constexpr int kFC = 8;    // frequencies per chunk of a spectrum
constexpr int kKT = 344;  // kernel values per frequency in khatT (343 offsets, padded)

template <int P>
constexpr int node_threads() { return (P * (P + 1) + 63) / 64 * 64; }

// Node of block g: the 8 XCDs (blocks dealt round robin) take contiguous runs
// of nodes, so that the [frequency][node] writes of neighbouring nodes meet in
// one L2.
__device__ __forceinline__ int64_t xcd_node(int64_t g, int64_t nn) { return (g & 7) * (nn >> 3) + (g >> 3); }

// Spectrum element (frequency f, node) of a level with nn nodes.
__device__ __forceinline__ int64_t sidx(int f, int64_t node, int64_t nn) {
  return ((int64_t)(f / kFC) * nn + node) * kFC + f % kFC;
}

// Forward transform of one node's p^3 gridlet (on the 2p cyclic grid, zero
// beyond p) to its half spectrum; frequency order
// ((kx * 2 + ky % 2) * p + ky / 2) * (p + 1) + kz.
// Spectra are stored as TS: double2, or float2 for the 16^3 leaf level
// summed in FP32 columns (half the bytes; its stencil rounds them to FP32
// anyway).
__device__ __forceinline__ double2 as_d2(double2 v) { return v; }
__device__ __forceinline__ double2 as_d2(float2 v) { return make_double2(v.x, v.y); }
template <class TS> __device__ __forceinline__ TS from_d2(double2 v);
template <> __device__ __forceinline__ double2 from_d2<double2>(double2 v) { return v; }
template <> __device__ __forceinline__ float2 from_d2<float2>(double2 v) {
  return make_float2((float)v.x, (float)v.y);
}

//
// load(i): mass i of the gridlet; A1, A2: P P (P + 1) values of LDS each; NT
// threads.  Ends with a barrier.
template <int P, int NT, class TS, class LOAD>
__device__ __forceinline__ void node_fwd_block(LOAD&& load, int64_t node, int64_t nn, TS* __restrict__ spec,
                                               double2* A1, double2* A2) {
  constexpr int M = 2 * P, H = P + 1;
  for (int r = threadIdx.x; r < P * P; r += NT) {
    double2 e[P], o[P];
#pragma unroll
    for (int z = 0; z < P; ++z) {
      e[z] = make_double2(load(r * P + z), 0.0);
      o[z] = dtwiddle<M, false>(e[z], z);
    }
    ddft<P, false>(e);
    ddft<P, false>(o);
    double2* row = A1 + r * H;
#pragma unroll
    for (int k = 0; k < H; ++k) row[k] = (k & 1) ? o[k >> 1] : e[k >> 1];
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    for (int r = threadIdx.x; r < P * H; r += NT) {
      const int x = r / H, kz = r % H;
      double2 u[P];
#pragma unroll
      for (int y = 0; y < P; ++y) {
        u[y] = A1[(x * P + y) * H + kz];
        if (h) u[y] = dtwiddle<M, false>(u[y], y);
      }
      ddft<P, false>(u);
#pragma unroll
      for (int m = 0; m < P; ++m) A2[(x * P + m) * H + kz] = u[m];
    }
    __syncthreads();
    for (int r = threadIdx.x; r < P * H; r += NT) {
      const int m = r / H, kz = r % H;
      double2 e[P], o[P];
#pragma unroll
      for (int x = 0; x < P; ++x) {
        e[x] = A2[(x * P + m) * H + kz];
        o[x] = dtwiddle<M, false>(e[x], x);
      }
      ddft<P, false>(e);
      ddft<P, false>(o);
#pragma unroll
      for (int j = 0; j < P; ++j) {
        spec[sidx((4 * j + h) * P * H + r, node, nn)] = from_d2<TS>(e[j]);
        spec[sidx((4 * j + 2 + h) * P * H + r, node, nn)] = from_d2<TS>(o[j]);
      }
    }
    __syncthreads();
  }
}

// Inverse of node_fwd_block at the p^3 gridlet points: store(i, v) takes point i;
// unnormalised (the kernel spectra carry 1 / (2p)^3).
template <int P, int NT, class TS, class STORE>
__device__ __forceinline__ void node_inv_block(const TS* __restrict__ spec, int64_t node, int64_t nn, double2* B1,
                                               double2* B2, STORE&& store) {
  constexpr int M = 2 * P, H = P + 1;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    for (int r = threadIdx.x; r < P * H; r += NT) {
      const int m = r / H, kz = r % H;
      double2 e[P], o[P];
#pragma unroll
      for (int j = 0; j < P; ++j) {
        e[j] = as_d2(spec[sidx((4 * j + h) * P * H + r, node, nn)]);
        o[j] = as_d2(spec[sidx((4 * j + 2 + h) * P * H + r, node, nn)]);
      }
      ddft<P, true>(e);
      ddft<P, true>(o);
#pragma unroll
      for (int x = 0; x < P; ++x) B1[(x * P + m) * H + kz] = dadd(e[x], dtwiddle<M, true>(o[x], x));
    }
    __syncthreads();
    for (int r = threadIdx.x; r < P * H; r += NT) {
      const int x = r / H, kz = r % H;
      double2 v[P];
#pragma unroll
      for (int m = 0; m < P; ++m) v[m] = B1[(x * P + m) * H + kz];
      ddft<P, true>(v);
#pragma unroll
      for (int y = 0; y < P; ++y) {
        double2& d = B2[(x * P + y) * H + kz];
        d = h ? dadd(d, dtwiddle<M, true>(v[y], y)) : v[y];
      }
    }
    __syncthreads();
  }
  for (int r = threadIdx.x; r < P * P; r += NT) {
    double2 u[H];
#pragma unroll
    for (int k = 0; k < H; ++k) u[k] = B2[r * H + k];
#pragma unroll
    for (int z = 0; z < P; ++z) {
      double b = 0.0;
#pragma unroll
      for (int k = 1; k < P; ++k) {
        const double2 w = twd<M>(k * z);
        b = fma(-u[k].y, w.y, fma(u[k].x, w.x, b));
      }
      const double v = fma(2.0, b, u[0].x + ((z & 1) ? -u[P].x : u[P].x));
      store(r * P + z, v);
    }
  }
}

}  // namespace
}  // namespace pfmm
