// The direct leaf near zone of single solves (the 27 neighbour leaves, Sec. 2),
// every sum in FP64, for leaf edges s = 4, 8, 16.
//
// Target leaf b, source leaf b + e, e in {-1, 0, 1}^3, cells c and c':
//   phi[b s + c] = h^3 sum_e sum_c' G(h (c - c' - s e)) rho[(b + e) s + c'].
// Each pair's separations c - c' have distinct residues on 2s points per axis,
// so the sums of a leaf pair are a cyclic convolution on the (2s)^3 grid, exact
// up to FP64 rounding (2^-53 times log s), and the 27 neighbours add per
// frequency: one forward transform per leaf, a 27-term sum at each of the
// (2s)^2 (s + 1) frequencies, one inverse per leaf and kernel.  The term-by-term
// sum, whose FP32 products cost 54 s^6 flops per leaf at 0.5 of the FP32 rate,
// takes (128^3, s = 16) 7.0 ms per kernel and 0.78 ms at 64^3, s = 8; this takes
// 0.157 and 0.034 ms (0.52 ms for the four kernels of the expansion accelerations
// against 28), and 1.21 ms at 256^3 against 45 in FP32 and 8 in split bf16 on the
// matrix cores.  Its error against 64 bits is that of
// rounding the result (4.5e-8 of the norm at 128^3; the FP32 sums 9.8e-7).  The
// transforms and sums are bound by HBM (144 B per cell of spectra, written and read
// twice) and, below 64 leaves an axis plane, by latency.
//
// Spectra are stored [frequency / 64][leaf][64] (1 KiB runs).  The leaf planes
// along x are swept in slabs whose source and target spectra fit in kSlabBytes:
// the forward transforms of a slab's planes and their two neighbours, then per
// kernel the sums and the inverse transforms of its planes.
#include "dft64.h"
#include "internal.h"

#include <algorithm>

namespace pfmm {

struct Near64 {
  int N = 0, s = 0, nb = 0, lgnb = 0;
  int F = 0;                 // (2s)^2 (s + 1) frequencies per leaf
  int ntabs = 0;             // kernels transformed so far
  int planes = 0;            // target leaf planes per slab (nb: the whole box, no slabs)
  int sources = 0;           // source leaf planes per slab
  double2* rhat = nullptr;   // spectra of the slab's source planes
  double2* yhat = nullptr;   // spectra of the slab's target planes (after rhat in one allocation)
  double2* khat[4] = {nullptr, nullptr, nullptr, nullptr};  // [F / 64][27][64] per kernel: the
                             // potential's after yhat, the accelerations' in an allocation of their own
  double2* tmp = nullptr;    // [27][F] between the passes of the kernels' transforms, which so touch
                             // neither spectra nor other kernels: solves that use those may be in flight
};

namespace {

constexpr int kThreads = 256;
constexpr int kMacWaves = 4;                    // waves of one workgroup of the sums (a power of two)
constexpr size_t kSlabBytes = (size_t)3 << 30;  // source and target spectra of a slab

inline unsigned nblk(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

// Threads per leaf: every pass has at most s (s + 1) tasks, one per thread.
template <int S>
constexpr int leaf_threads() { return (S * (S + 1) + 63) / 64 * 64; }

// Frequency f of leaf slot `leaf` among nl slots.
__device__ __forceinline__ int64_t at64(int f, int64_t leaf, int64_t nl) {
  return ((int64_t)(f >> 6) * nl + leaf) * 64 + (f & 63);
}

// Rows of S values of the mesh, 16 bytes at a time when the array allows.
template <int S>
__device__ __forceinline__ void load_row(const float* src, bool vec, double (&v)[S]) {
  if (vec) {
#pragma unroll
    for (int q = 0; q < S / 4; ++q) {
      const float4 a = reinterpret_cast<const float4*>(src)[q];
      v[4 * q] = a.x;
      v[4 * q + 1] = a.y;
      v[4 * q + 2] = a.z;
      v[4 * q + 3] = a.w;
    }
  } else {
#pragma unroll
    for (int z = 0; z < S; ++z) v[z] = src[z];
  }
}
template <int S>
__device__ __forceinline__ void load_row(const double* src, bool vec, double (&v)[S]) {
  if (vec) {
#pragma unroll
    for (int q = 0; q < S / 2; ++q) {
      const double2 a = reinterpret_cast<const double2*>(src)[q];
      v[2 * q] = a.x;
      v[2 * q + 1] = a.y;
    }
  } else {
#pragma unroll
    for (int z = 0; z < S; ++z) v[z] = src[z];
  }
}
template <int S>
__device__ __forceinline__ void store_row(float* dst, bool vec, const double (&v)[S]) {
  if (vec) {
#pragma unroll
    for (int q = 0; q < S / 4; ++q)
      reinterpret_cast<float4*>(dst)[q] =
          make_float4((float)v[4 * q], (float)v[4 * q + 1], (float)v[4 * q + 2], (float)v[4 * q + 3]);
  } else {
#pragma unroll
    for (int z = 0; z < S; ++z) dst[z] = (float)v[z];
  }
}
template <int S>
__device__ __forceinline__ void store_row(double* dst, bool vec, const double (&v)[S]) {
  if (vec) {
#pragma unroll
    for (int q = 0; q < S / 2; ++q) reinterpret_cast<double2*>(dst)[q] = make_double2(v[2 * q], v[2 * q + 1]);
  } else {
#pragma unroll
    for (int z = 0; z < S; ++z) dst[z] = v[z];
  }
}

// Forward transform of one leaf (zero beyond s on every axis) to its half
// spectrum, frequency ((kx * 2 + ky % 2) * s + ky / 2) * (s + 1) + kz.  Every
// pass splits its 2s outputs by parity into two DFTs of length s,
// X[2m] = DFT(u)[m] and X[2m + 1] = DFT(u_n w^n)[m].  The work runs once per
// parity of ky in one LDS buffer of s^2 (s + 1) values (68 KiB at s = 16, two
// leaves per CU): the z pass fills it from the row each thread keeps in
// registers, the y pass transforms the columns in place, the x pass reads it
// out, each parity of kx in turn.
template <int S, class TIN>
__global__ void __launch_bounds__(leaf_threads<S>()) k_fwd64(const TIN* __restrict__ rho, int N, int lgnb,
                                                             int plane0, int64_t nl, int vec,
                                                             double2* __restrict__ rhat) {
  constexpr int M = 2 * S, H = S + 1;
  __shared__ double2 A[S * S * H];
  const int64_t leaf = xcd_leaf(blockIdx.x, gridDim.x);  // slot: planes from plane0 on, wrapped
  const int msk = (1 << lgnb) - 1;
  const int bz = (int)(leaf & msk), by = (int)((leaf >> lgnb) & msk);
  const int bx = (plane0 + (int)(leaf >> (2 * lgnb))) & msk;
  const int tr = threadIdx.x;
  double row[S];
  if (tr < S * S)
    load_row<S>(rho + ((int64_t)(bx * S + tr / S) * N + (by * S + tr % S)) * N + (int64_t)bz * S, vec != 0, row);
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    if (tr < S * S) {
      double2* dst = A + tr * H;
      double2 v[S];
#pragma unroll
      for (int z = 0; z < S; ++z) v[z] = make_double2(row[z], 0.0);
      ddft<S, false>(v);
#pragma unroll
      for (int m = 0; m <= S / 2; ++m) dst[2 * m] = v[m];
#pragma unroll
      for (int z = 0; z < S; ++z) v[z] = dtwiddle<M, false>(make_double2(row[z], 0.0), z);
      ddft<S, false>(v);
#pragma unroll
      for (int m = 0; m < S / 2; ++m) dst[2 * m + 1] = v[m];
    }
    __syncthreads();
    if (tr < S * H) {
      double2* col = A + (tr / H) * S * H + tr % H;
      double2 u[S];
#pragma unroll
      for (int y = 0; y < S; ++y) {
        u[y] = col[y * H];
        if (h) u[y] = dtwiddle<M, false>(u[y], y);
      }
      ddft<S, false>(u);
#pragma unroll
      for (int m = 0; m < S; ++m) col[m * H] = u[m];
    }
    __syncthreads();
    if (tr < S * H) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        double2 u[S];
#pragma unroll
        for (int x = 0; x < S; ++x) {
          u[x] = A[x * S * H + tr];
          if (c) u[x] = dtwiddle<M, false>(u[x], x);
        }
        ddft<S, false>(u);
#pragma unroll
        for (int j = 0; j < S; ++j) rhat[at64(((2 * j + c) * 2 + h) * S * H + tr, leaf, nl)] = u[j];
      }
    }
    __syncthreads();
  }
}

// Inverse of k_fwd64 at the s^3 target cells of one leaf, written into the
// mesh (unnormalised: the kernels carry 1 / (2s)^3): per parity of ky the x
// pass v[x] = IDFT(Y_even)[x] + exp(2 pi i x / 2s) IDFT(Y_odd)[x] fills the
// buffer and the thread of each (x, kz) column does its y pass; the first
// parity's result waits in registers and the second parity's sum goes back in
// place for the real inverse along z.
template <int S, class TOUT>
__global__ void __launch_bounds__(leaf_threads<S>()) k_inv64(const double2* __restrict__ yhat, int N, int lgnb,
                                                             int plane0, int64_t nl, int vec,
                                                             TOUT* __restrict__ out) {
  constexpr int M = 2 * S, H = S + 1;
  __shared__ double2 B[S * S * H];
  const int64_t leaf = xcd_leaf(blockIdx.x, gridDim.x);
  const int msk = (1 << lgnb) - 1;
  const int bz = (int)(leaf & msk), by = (int)((leaf >> lgnb) & msk), bx = plane0 + (int)(leaf >> (2 * lgnb));
  const int tr = threadIdx.x;
  double2 acc[S];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (tr < S * H) {
      double2 e[S];
#pragma unroll
      for (int j = 0; j < S; ++j) e[j] = yhat[at64((4 * j + h) * S * H + tr, leaf, nl)];
      ddft<S, true>(e);
#pragma unroll
      for (int x = 0; x < S; ++x) B[x * S * H + tr] = e[x];
#pragma unroll
      for (int j = 0; j < S; ++j) e[j] = yhat[at64((4 * j + 2 + h) * S * H + tr, leaf, nl)];
      ddft<S, true>(e);
#pragma unroll
      for (int x = 0; x < S; ++x) B[x * S * H + tr] = dadd(B[x * S * H + tr], dtwiddle<M, true>(e[x], x));
    }
    __syncthreads();
    if (tr < S * H) {
      double2* col = B + (tr / H) * S * H + tr % H;
      double2 v[S];
#pragma unroll
      for (int m = 0; m < S; ++m) v[m] = col[m * H];
      ddft<S, true>(v);
#pragma unroll
      for (int y = 0; y < S; ++y) {
        if (h == 0)
          acc[y] = v[y];
        else
          col[y * H] = dadd(acc[y], dtwiddle<M, true>(v[y], y));
      }
    }
    __syncthreads();
  }
  if (tr < S * S) {
    double v[S];
    const double2* u = B + tr * H;
#pragma unroll
    for (int z = 0; z < S; ++z) v[z] = u[0].x + ((z & 1) ? -u[S].x : u[S].x);
#pragma unroll
    for (int k = 1; k < S; ++k) {
      const double2 y = make_double2(2.0 * u[k].x, 2.0 * u[k].y);
#pragma unroll
      for (int z = 0; z < S; ++z) {
        const double2 w = twd<M>(k * z);
        v[z] = fma(y.x, w.x, v[z]);
        v[z] = fma(-y.y, w.y, v[z]);
      }
    }
    store_row<S>(out + ((int64_t)(bx * S + tr / S) * N + (by * S + tr % S)) * N + (int64_t)bz * S, vec != 0, v);
  }
}

// yhat_b(k) = sum_e khat_e(k) rhat_{b+e}(k): a lane owns one frequency of a
// chunk and a 2 x 2 block of leaf pencils, swept along a segment of z.  Each step reads one
// z-plane of the 4 x 4 source columns around the block (16 bytes a lane, 1 KiB
// a wave; four reads an output) and adds it to the three target planes that
// see it, so one source plane and three planes of sums are in registers.  The
// 27 kernel values of a frequency are in LDS, shared by the kMacWaves waves of
// a workgroup, which take neighbouring blocks or segments (their number is a
// multiple of it: at least two by two blocks).  The pencil blocks of one chunk
// run on one XCD, whose L2 serves the columns they share.
//
// Bound: waiting for memory (three or four waves a SIMD; 284 MB in 85 us at 128^3,
// s = 16).  One wave a workgroup, its 27 KiB of kernel values its own, left 1.25
// waves a SIMD, and a branch around every load one load in flight: 125 us at
// 128^3, 29 (17 now) at 64^3, s = 8, 860 (610) at 256^3.  A second source plane in flight
// took more registers and was slower (the whole near zone at 128^3 165 against 157 us).
//
// Target planes x0 .. x0 + nx - 1 (nx even, slots from 0 in yhat); source plane x sits
// in slot (x - xs) mod nb of rhat (xs = 0 and nb slots without slabs).
template <bool ISO>
__global__ void __launch_bounds__(64 * kMacWaves, 3) k_mac64(const double2* __restrict__ rhat, const double2* __restrict__ khat,
                                              int nb, int nchunk, int x0, int nx, int xs, int nz,
                                              int64_t nls, int64_t nlt, double2* __restrict__ yhat) {
  __shared__ double2 kks[27 * 64];
  const int hy = nb >> 1, hz = nb / nz, np = (nx >> 1) * hy * hz;  // 2 x 2 pencil blocks, z segments
  const int j = blockIdx.x >> 3, ng = np / kMacWaves;              // groups of kMacWaves of them
  const int chunk = (j / ng) * 8 + (blockIdx.x & 7);
  if (chunk >= nchunk) return;
  const int lane = threadIdx.x & 63, msk = nb - 1;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blk = j % ng * kMacWaves + wave;
  const int bx0 = x0 + 2 * (blk / (hy * hz)), by0 = 2 * ((blk / hz) % hy), z0 = blk % hz * nz;
  const double2* src = rhat + (int64_t)chunk * nls * 64 + lane;
  double2* dst = yhat + (int64_t)chunk * nlt * 64 + lane;
  double2* kk = kks + lane;
  for (int e = wave; e < 27; e += kMacWaves) kk[e * 64] = khat[((int64_t)chunk * 27 + e) * 64 + lane];
  __syncthreads();
  unsigned col[16];  // source columns (bx0 - 1 + ix, by0 - 1 + iy), c = 4 ix + iy
  bool in[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const int sx = bx0 - 1 + c / 4, sy = by0 - 1 + c % 4;
    in[c] = !ISO || (sx >= 0 && sx < nb && sy >= 0 && sy < nb);
    col[c] = (unsigned)((((sx & msk) - xs) & msk) * nb + (sy & msk)) * nb;
    if (ISO && !in[c]) col[c] = 0;  // any slot (its column may not be in the slab)
  }
  const double2 zero = make_double2(0.0, 0.0);
  auto load_plane = [&](double2 (&v)[16], int z) {
    const bool zin = !ISO || (z >= 0 && z < nb);
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      v[c] = src[(int64_t)(col[c] + (unsigned)(z & msk)) * 64];
      if (ISO && !(zin && in[c])) v[c] = zero;
    }
  };
  struct Sums {
    double2 t[4];
  };
  // source plane z, the neighbour ez - 1 of target plane z + 1 - ez
  auto plane = [&](const double2 (&v)[16], Sums& s, int ez) {
#pragma unroll
    for (int ex = 0; ex < 3; ++ex)
#pragma unroll
      for (int ey = 0; ey < 3; ++ey) {
        // kernel values are read here every time, not kept in registers
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        const double2 k = kk[(ex * 9 + ey * 3 + ez) * 64];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const double2 q = v[(t / 2 + ex) * 4 + t % 2 + ey];
          s.t[t].x = fma(k.x, q.x, s.t[t].x);
          s.t[t].x = fma(-k.y, q.y, s.t[t].x);
          s.t[t].y = fma(k.x, q.y, s.t[t].y);
          s.t[t].y = fma(k.y, q.x, s.t[t].y);
        }
      }
  };
  double2 v[16];
  Sums s0, s1, s2;
  // source plane z; `lo`, `mid`, `up` are the sums of the target planes z - 1, z, z + 1
  auto step = [&](int z, Sums& lo, Sums& mid, Sums& up, bool do_lo, bool do_mid, bool do_up) {
    load_plane(v, z);
    if (do_lo) {
      plane(v, lo, 2);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        dst[((int64_t)((bx0 - x0 + t / 2) * nb + by0 + t % 2) * nb + z - 1) * 64] = lo.t[t];
    }
    if (do_mid) plane(v, mid, 1);
    if (do_up) {
#pragma unroll
      for (int t = 0; t < 4; ++t) up.t[t] = zero;
      plane(v, up, 0);
    }
  };
  const int zl = z0 + nz - 1;
  step(z0 - 1, s1, s2, s0, false, false, true);
  step(z0, s2, s0, s1, false, true, true);
#pragma unroll 1
  for (int z = z0 + 1; z < zl; z += 2) {  // nz is even
    step(z, s0, s1, s2, true, true, true);
    step(z + 1, s1, s2, s0, true, true, true);
    s1 = s0;
    s0 = s2;
  }
  step(zl, s0, s1, s2, true, true, false);
  step(zl + 1, s1, s2, s0, true, false, false);
}

// Kernel transforms, neighbour e = blockIdx.y of K_e[m] = tab[m - s e] (tab
// centred, edge 4s - 1; the unused slot m = s is zero): along z, then y, x.
__device__ __forceinline__ void twiddles(int M, double2* w) {  // exp(-2 pi i j / M)
  for (int j = threadIdx.x; j < M; j += kThreads) sincospi(-2.0 * j / M, &w[j].y, &w[j].x);
  __syncthreads();
}

__global__ void k_kz64(const double* __restrict__ tab, int s, double2* __restrict__ out) {
  __shared__ double2 w[32];
  const int M = 2 * s, H = s + 1, C = 2 * s - 1, E = 2 * C + 1;
  twiddles(M, w);
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= M * M * H) return;
  const int ex = blockIdx.y / 9 - 1, ey = (blockIdx.y / 3) % 3 - 1, ez = blockIdx.y % 3 - 1;
  const int kz = i % H, y = (i / H) % M, x = i / (H * M);
  double re = 0.0, im = 0.0;
  if (x != s && y != s) {
    const int jx = (x < s ? x : x - M) - s * ex, jy = (y < s ? y : y - M) - s * ey;
    const double* row = tab + ((int64_t)(jx + C) * E + (jy + C)) * E + C - s * ez;
    for (int z = 0; z < M; ++z) {
      if (z == s) continue;
      const double v = row[z < s ? z : z - M];
      const double2 t = w[(kz * z) & (M - 1)];
      re = fma(v, t.x, re);
      im = fma(v, t.y, im);
    }
  }
  out[(int64_t)blockIdx.y * M * M * H + i] = make_double2(re, im);
}

// Pass along y (axis 1) into the same layout, or along x (axis 0), scaled, into
// [F / 64][27][64] in the frequency order of k_fwd64.
__global__ void k_kaxis64(const double2* __restrict__ in, int s, int axis, double scale,
                          double2* __restrict__ out) {
  __shared__ double2 w[32];
  const int M = 2 * s, H = s + 1, F = M * M * H;
  twiddles(M, w);
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= F) return;
  in += (int64_t)blockIdx.y * F;
  const int kz = i % H, b = (i / H) % M, a = i / (H * M);
  const int k = axis ? b : a, step = axis ? H : M * H;
  const double2* src = in + (axis ? a * M * H + kz : b * H + kz);
  double re = 0.0, im = 0.0;
  for (int j = 0; j < M; ++j) {
    const double2 v = src[j * step], t = w[(k * j) & (M - 1)];
    re += v.x * t.x - v.y * t.y;
    im += v.x * t.y + v.y * t.x;
  }
  if (axis) {
    out[(int64_t)blockIdx.y * F + i] = make_double2(re, im);
  } else {
    const int f = ((a * 2 + (b & 1)) * s + (b >> 1)) * H + kz;  // kx = a, ky = b
    out[((int64_t)(f >> 6) * 27 + blockIdx.y) * 64 + (f & 63)] = make_double2(re * scale, im * scale);
  }
}

template <class T>
bool aligned16(const T* p) { return ((uintptr_t)p & 15) == 0; }

template <class TIN>
hipError_t fwd_any(const Near64* f, const TIN* rho, int plane0, int planes, hipStream_t st) {
  const unsigned blocks = (unsigned)planes * f->nb * f->nb;
  const int64_t nl = blocks;
  const int vec = aligned16(rho);
  if (f->s == 4)
    k_fwd64<4, TIN><<<blocks, leaf_threads<4>(), 0, st>>>(rho, f->N, f->lgnb, plane0, nl, vec, f->rhat);
  else if (f->s == 8)
    k_fwd64<8, TIN><<<blocks, leaf_threads<8>(), 0, st>>>(rho, f->N, f->lgnb, plane0, nl, vec, f->rhat);
  else
    k_fwd64<16, TIN><<<blocks, leaf_threads<16>(), 0, st>>>(rho, f->N, f->lgnb, plane0, nl, vec, f->rhat);
  return hipGetLastError();
}

template <class TOUT>
hipError_t inv_any(const Near64* f, TOUT* out, int plane0, int planes, hipStream_t st) {
  const unsigned blocks = (unsigned)planes * f->nb * f->nb;
  const int64_t nl = blocks;
  const int vec = aligned16(out);
  if (f->s == 4)
    k_inv64<4, TOUT><<<blocks, leaf_threads<4>(), 0, st>>>(f->yhat, f->N, f->lgnb, plane0, nl, vec, out);
  else if (f->s == 8)
    k_inv64<8, TOUT><<<blocks, leaf_threads<8>(), 0, st>>>(f->yhat, f->N, f->lgnb, plane0, nl, vec, out);
  else
    k_inv64<16, TOUT><<<blocks, leaf_threads<16>(), 0, st>>>(f->yhat, f->N, f->lgnb, plane0, nl, vec, out);
  return hipGetLastError();
}

template <class T>
hipError_t run(const Near64* f, const T* rho, T* const* out, int nout, int isolated, hipStream_t st) {
  const int nb = f->nb, nchunk = f->F / 64;
  const bool whole = f->planes >= nb;
  hipError_t e = hipSuccess;
  for (int x0 = 0; x0 < nb && e == hipSuccess; x0 += f->planes) {
    const int nx = std::min(f->planes, nb - x0);
    const int xs = whole ? 0 : x0 - 1, ns = whole ? nb : nx + 2;  // source planes xs .. xs + ns - 1
    e = fwd_any(f, rho, xs & (nb - 1), ns, st);
    const int64_t nls = (int64_t)ns * nb * nb, nlt = (int64_t)nx * nb * nb;
    // whole pencils unless that leaves the SIMDs (4 a CU) idle: a segment reads
    // two more planes than it writes
    unsigned waves = (unsigned)((nchunk + 7) / 8 * 8) * (unsigned)(nx / 2) * (unsigned)(nb / 2);
    int nz = nb;
    for (; nz > 2 && waves < 2048; nz /= 2) waves *= 2;
    const unsigned blocks = waves / kMacWaves;
    for (int t = 0; t < nout && e == hipSuccess; ++t) {
      if (isolated)
        k_mac64<true><<<blocks, 64 * kMacWaves, 0, st>>>(f->rhat, f->khat[t], nb, nchunk, x0, nx,
                                             xs & (nb - 1), nz, nls, nlt, f->yhat);
      else
        k_mac64<false><<<blocks, 64 * kMacWaves, 0, st>>>(f->rhat, f->khat[t], nb, nchunk, x0, nx,
                                             xs & (nb - 1), nz, nls, nlt, f->yhat);
      e = hipGetLastError();
      if (e == hipSuccess) e = inv_any(f, out[t], x0, nx, st);
    }
  }
  return e;
}

}  // namespace

void near64_destroy(Near64* f) {
  if (!f) return;
  (void)hipFree(f->rhat);
  (void)hipFree(f->khat[1]);
  delete f;
}

namespace {
// The sizes of the buffers, and the bytes they take.
size_t shape(int N, int s, Near64* f) {
  f->N = N;
  f->s = s;
  f->nb = N / s;
  while ((1 << f->lgnb) < f->nb) ++f->lgnb;
  f->F = 4 * s * s * (s + 1);
  const int nb = f->nb;
  const size_t plane = (size_t)nb * nb * f->F;
  // the whole box, or slabs of an even number of planes (at least two) with
  // their two neighbours
  f->planes = nb;
  if (2 * (size_t)nb * plane * sizeof(double2) > kSlabBytes) {
    const size_t fit = kSlabBytes / (plane * sizeof(double2));
    f->planes = fit >= 6 ? (int)((fit - 2) / 2 & ~(size_t)1) : 2;
    if (f->planes + 2 >= nb) f->planes = nb;
  }
  f->sources = f->planes == nb ? nb : f->planes + 2;
  return ((size_t)(f->sources + f->planes) * plane + (size_t)54 * f->F) * sizeof(double2);
}
}  // namespace

size_t near64_bytes(int N, int s) {
  Near64 f;
  return shape(N, s, &f);
}

hipError_t near64_create(int N, int s, Near64** out) {
  *out = nullptr;
  if (s != 4 && s != 8 && s != 16) return hipErrorInvalidValue;
  Near64* f = new Near64;
  const hipError_t e = hipMalloc(&f->rhat, shape(N, s, f));
  if (e != hipSuccess) {
    near64_destroy(f);
    return e;
  }
  const size_t plane = (size_t)f->nb * f->nb * f->F;
  f->yhat = f->rhat + f->sources * plane;
  f->khat[0] = f->yhat + f->planes * plane;
  f->tmp = f->khat[0] + (size_t)27 * f->F;
  *out = f;
  return hipSuccess;
}

hipError_t near64_tables(Near64* f, const double* const* tabs, int first, int ntabs, double scale,
                         hipStream_t st) {
  if (first < 0 || ntabs < 1 || ntabs > 4) return hipErrorInvalidValue;
  const double sc = scale / (8.0 * f->s * f->s * f->s);  // the inverse transform is unnormalised
  const dim3 grid(nblk(f->F), 27);
  const size_t one = (size_t)27 * f->F;
  hipError_t e = hipSuccess;
  if (ntabs > 1 && !f->khat[1]) {
    double2* k = nullptr;
    e = hipMalloc(&k, 3 * one * sizeof(double2));
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      e = hipSuccess;
      ntabs = 1;
    } else if (e != hipSuccess) {
      return e;
    } else {
      for (int t = 1; t < 4; ++t) f->khat[t] = k + (t - 1) * one;
    }
  }
  for (int t = first; t < ntabs && e == hipSuccess; ++t) {
    k_kz64<<<grid, kThreads, 0, st>>>(tabs[t], f->s, f->khat[t]);
    k_kaxis64<<<grid, kThreads, 0, st>>>(f->khat[t], f->s, 1, 1.0, f->tmp);
    k_kaxis64<<<grid, kThreads, 0, st>>>(f->tmp, f->s, 0, sc, f->khat[t]);
    e = hipGetLastError();
  }
  f->ntabs = e == hipSuccess ? std::max(f->ntabs, ntabs) : 0;
  return e;
}

int near64_kernels(const Near64* f) { return f ? f->ntabs : 0; }

hipError_t near64_run(const Near64* f, const float* rho, float* const* out, int nout, int isolated,
                      hipStream_t st) {
  return nout < 1 || nout > f->ntabs ? hipErrorInvalidValue : run(f, rho, out, nout, isolated, st);
}

hipError_t near64_run_f64(const Near64* f, const double* rho, double* const* out, int nout, int isolated,
                          hipStream_t st) {
  return nout < 1 || nout > f->ntabs ? hipErrorInvalidValue : run(f, rho, out, nout, isolated, st);
}

}  // namespace pfmm
