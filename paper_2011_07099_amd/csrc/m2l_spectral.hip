// Interaction zones (Eq. 6) as spectral stencils over the nodes of a level.
//
// Target node t, source node t + d (d in the zone of t's parity class, 189
// offsets at levels >= 3; the periodic level-2 zone), gridlet points a, a':
//   Phi_l[t][a] += sum_d sum_a' G(eta_l (a - a' - p d)) M_l[t + d][a'].
// For one d this is a linear convolution of a p^3 block with the kernel
// K_d[m] = G(eta_l (m - p d)), |m_i| <= p - 1, so, as for the leaf near zone,
// it is exact as a cyclic convolution on 2p points per axis, and the zone's
// offsets add per frequency:
//   Phi_hat_t(k) = sum_{d in IZ(t)} K_hat_d(k) M_hat_{t+d}(k).
// One forward transform per node, a stencil of 189 (37 at level 2) terms per
// target and frequency, one inverse per node.  Against the block-Toeplitz
// GEMM's 2 p^6 flops per target and offset this is 8 flops per frequency
// ((2p)^2 (p + 1) of them) plus the transforms.
//
// Everything here is FP64 (transforms, kernel spectra, stencil); masses are read
// and potentials added in the level's own precision.  Kernel spectra (all 343
// offsets of [-3, 3]^3) are transformed once per table.  PFMM_M2L_SPECTRAL and
// most levels of the default zones run this way.
//
// Layout: spectra of a level as [frequency / 8][node][frequency % 8]: a
// node's transform writes (and its inverse reads) 128-byte runs, and the 8
// frequencies of a chunk, whose stencil workgroups run on one XCD, share
// every line of it.
#include "spectral.h"

#include <algorithm>

namespace pfmm {

namespace {

constexpr int kThreads = 256;
inline unsigned nblk(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

template <int P, class TIN, class TS = double2>
__global__ void __launch_bounds__(node_threads<P>()) k_node_fwd(const TIN* __restrict__ Ml, int64_t nn,
                                                                TS* __restrict__ spec) {
  __shared__ double2 A1[P * P * (P + 1)];
  __shared__ double2 A2[P * P * (P + 1)];
  const int64_t node = xcd_node(blockIdx.x, nn);
  const TIN* src = Ml + node * (P * P * P);
  node_fwd_block<P, node_threads<P>()>([&](int i) { return (double)src[i]; }, node, nn, spec, A1, A2);
}

// Added to (or written into) the node's potentials.
template <int P, class TOUT, class TS = double2>
__global__ void __launch_bounds__(node_threads<P>()) k_node_inv(const TS* __restrict__ spec,
                                                                int64_t nn, int accumulate,
                                                                TOUT* __restrict__ Pl) {
  __shared__ double2 B1[P * P * (P + 1)];
  __shared__ double2 B2[P * P * (P + 1)];
  const int64_t node = xcd_node(blockIdx.x, nn);
  TOUT* dst = Pl + node * (P * P * P);
  node_inv_block<P, node_threads<P>()>(spec, node, nn, B1, B2, [&](int i, double v) {
    dst[i] = accumulate ? (TOUT)((double)dst[i] + v) : (TOUT)v;
  });
}

// (re, im) += k s, one complex multiply-add as four FMAs
__device__ __forceinline__ void cmac(double& re, double& im, double2 k, double2 s) {
  re = fma(k.x, s.x, re);
  re = fma(-k.y, s.y, re);
  im = fma(k.x, s.y, im);
  im = fma(k.y, s.x, im);
}
// A wave-uniform FP32 value copied into a vector register, so that the
// multiply-adds that use it take the two-operand form with all operands in
// vector registers, which gfx950 issues at twice the rate of the forms with
// a scalar operand or a negation modifier.
__device__ __forceinline__ float vreg(float x) {
  float r;
  asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(x));
  return r;
}

template <class T> struct Vec2;
template <> struct Vec2<double> { using type = double2; };
template <> struct Vec2<float> { using type = float2; };

// The 16 x 16 x 4 FP64 matrix-core product d += a b.  Operands: lane l holds
// a[l % 16][l / 16] and b[l / 16][l % 16].  Results: lane l holds column l % 16
// of the rows 4 r + l / 16, in register r.
typedef double v4d __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4d mma(double a, double b, v4d d) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d, 0, 0, 0);
}

// The zones of a level as matrix products over octets.  The eight targets of
// one parent see together the 6^3 children of the parent's 27 neighbours
// (Sec. 2), s_i in [-2, 3] counted from the parent's first child; the pair
// (source s, target t) is in the zone unless every |s_i - t_i| <= 1, and its
// kernel is that of d = s - t.  So at one frequency the targets of all parents
// are one product, complex [8 x 216] by [216 x parents], 189 / 216 of whose
// kernel entries are in the zone (the others are zero): real
// [16 x 432] by [432 x parents] with the rows (target, re / im), the columns
// (source, re / im) and [re, -im; im, re] blocks, on the matrix cores in steps
// of four columns (two sources neighbouring in z).  Both operands are read
// from LDS at one address per lane plus a constant: the kernel's entry index
// is linear in s and in t, the sources are split by child,
// [px][py][pz][hx][hy][hz], where a step of s moves whole parents.
//
// One workgroup per (frequency, tile of HX x HY x HZ parents); a wave sums G
// groups of 16 parents, which share the kernel operand.  WRAP: the tile is the
// whole periodic level and parents wrap.  Else the tile has a halo of one
// parent (wrapped, or zero outside an isolated box).
//
// Bound: the matrix cores (108 products of 64 cycles, FP64, per 16 parents and
// frequency; they are busy 0.57-0.67 of the kernel) plus the staging, whose
// 16-byte reads at a 128-byte stride do not all hide behind the products.  On
// the vector ALUs, one lane per target and parity class, LDS reads (one per
// multiply-add) and waits for scalar kernel loads were the bound.  Measured,
// p = 8, before / after: 32^3 level 4.23 / 2.72 ms (1.14e11 flops), 8^3 level
// 59 / 49 us, isolated 16^3 level at p = 4 77 / 55 us; the periodic 16^3 level
// would take 330 us here against the 325 us of the runs along y below, which
// keep it.  The same octets on the vector ALUs (kernel values by scalar loads)
// took 2.6-2.9 ms and 57 us: as fast at 32^3, slower at 8^3, where a wave waits
// for its scalar loads.
template <int HX, int HY, int HZ, int G, bool WRAP>
__global__ void __launch_bounds__(HX * HY * HZ * 4 / G, 4) k_zone_oct(
    const double2* __restrict__ spec, const double2* __restrict__ khatT, int n, int isolated,
    int nchunk, double2* __restrict__ out) {
  constexpr int NP = HX * HY * HZ, NT = NP * 4 / G, HALO = WRAP ? 0 : 1;
  constexpr int BX = HX + 2 * HALO, BY = HY + 2 * HALO, BZ = HZ + 2 * HALO, B3 = BX * BY * BZ;
  static_assert(16 % HZ == 0 && (HY * HZ) % (16 * G) == 0, "a wave's groups share h_x, its lanes h_z");
  __shared__ double2 box[8 * B3];
  // kernel entry (dx, dy, dz) at (dx + 3) KX + (dy + 3) 7 + dz + 3: with planes
  // of 51 entries the 8 targets' entries fall on different banks
  constexpr int KX = 51;
  __shared__ double2 kk[7 * KX];
  const int hn = n >> 1;  // parents per axis
  const int tpx = hn / HX, tpy = hn / HY, tpz = hn / HZ, tiles = tpx * tpy * tpz;
  // the 8 XCDs (blocks dealt round robin) take whole chunks, a tile's kFC
  // frequencies, which share their lines, back to back
  const int blk = blockIdx.x >> 3;
  const int chunk = (blk / (kFC * tiles)) * 8 + (blockIdx.x & 7);
  if (chunk >= nchunk) return;
  const int f = blk % kFC, tile = (blk / kFC) % tiles;
  const int ox = (tile / (tpy * tpz)) * HX, oy = ((tile / tpz) % tpy) * HY, oz = (tile % tpz) * HZ;
  const int64_t nn = (int64_t)n * n * n;
  const double2* sk = spec + (int64_t)chunk * nn * kFC + f;  // node v at sk[kFC v]
  for (int i = threadIdx.x; i < 8 * B3; i += NT) {
    const int bz = i % (2 * BZ), by = (i / (2 * BZ)) % (2 * BY), bx = i / (4 * BZ * BY);
    const int x = 2 * (ox - HALO) + bx, y = 2 * (oy - HALO) + by, z = 2 * (oz - HALO) + bz;
    double2 v = make_double2(0.0, 0.0);
    if (WRAP || !isolated ||
        ((unsigned)x < (unsigned)n && (unsigned)y < (unsigned)n && (unsigned)z < (unsigned)n))
      v = sk[(((int64_t)(x & (n - 1)) * n + (y & (n - 1))) * n + (z & (n - 1))) * kFC];
    box[(((bx & 1) * 2 + (by & 1)) * 2 + (bz & 1)) * B3 + ((bx >> 1) * BY + (by >> 1)) * BZ + (bz >> 1)] = v;
  }
  for (int i = threadIdx.x; i < 343; i += NT) {
    const int dx = i / 49 - 3, dy = (i / 7) % 7 - 3, dz = i % 7 - 3;
    const bool near = abs(dx) <= 1 && abs(dy) <= 1 && abs(dz) <= 1;
    kk[(dx + 3) * KX + i % 49] = near ? make_double2(0.0, 0.0) : khatT[(int64_t)(chunk * kFC + f) * kKT + i];
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15;                              // row of a, column of b
  const int cs = (lane >> 4) & 1, pz = lane >> 5;         // step column: source component and z child
  // a's row: target t = (tx, ty, tz) = (reg / 2, quad / 2, quad % 2), component reg % 2
  const int ra = col >> 2, qa = col & 3;
  const double* ka = &kk[0].x + (((3 - (ra >> 1)) * KX + (3 - (qa >> 1)) * 7 + 3 - (qa & 1) + pz) * 2 + ((ra & 1) ^ cs));
  const bool neg = (ra & 1) == 0 && cs == 1;              // -im in the real rows
  // b's column: a parent of each group
  const int p0 = wave * G * 16;
  const int hx = p0 / (HY * HZ), hz = col % HZ;
  auto at = [](int h, int q, int H) { return WRAP ? (h + q) & (H - 1) : h + q + 1; };  // parent h + q
  int zi[3], yi[G][3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    zi[q] = (pz * B3 + at(hz, q - 1, HZ)) * 2 + cs;
#pragma unroll
    for (int g = 0; g < G; ++g) yi[g][q] = at((p0 / HZ + (g * 16 + col) / HZ) % HY, q - 1, HY) * (BZ * 2);
  }
  v4d acc[G];
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = v4d{0.0, 0.0, 0.0, 0.0};
  for (int sx = -2; sx <= 3; ++sx) {
    const double* bx = &box[0].x + ((sx & 1) * 4 * B3 + at(hx, sx >> 1, HX) * BY * BZ) * 2;
    const double* kx = ka + sx * (2 * KX);
#pragma unroll
    for (int sy = -2; sy <= 3; ++sy) {
      const double* by = bx + (sy & 1) * 4 * B3;
#pragma unroll
      for (int m = 0; m < 3; ++m) {  // sources s_z = 2 m - 2, 2 m - 1
        double a = kx[sy * 14 + (2 * m - 2) * 2];
        a = neg ? -a : a;
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = mma(a, by[yi[g][(sy >> 1) + 1] + zi[m]], acc[g]);
      }
    }
  }
  double2* o = out + (int64_t)chunk * nn * kFC + f;
  const int q = lane >> 4;  // results: target (reg / 2, q / 2, q % 2), component reg % 2
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int hy = (p0 / HZ + (g * 16 + col) / HZ) % HY;
#pragma unroll
    for (int tx = 0; tx < 2; ++tx) {
      const int x = 2 * (ox + hx) + tx, y = 2 * (oy + hy) + (q >> 1), z = 2 * (oz + hz) + (q & 1);
      o[(((int64_t)x * n + y) * n + z) * kFC] = make_double2(acc[g][2 * tx], acc[g][2 * tx + 1]);
    }
  }
}

// Whole-level stencil, targets in runs along y (used for the 16^3 level, n =
// 2H = 16): one workgroup per frequency holds the level's whole spectrum at that
// frequency in LDS (n^3 values: periodic wrap, no halo) and sums every
// target's zone.  Stored split by parity, [px][py][pz][hx][hy][hz] (node
// coordinate 2h + p), hz fastest.  With H = 8 and TY = 8 one wave per
// parity class: the class, the zone's offsets and so every kernel value are
// uniform across a wave, and the kernel values come from the frequency's
// contiguous row of khatT by scalar loads, leaving LDS to the sources.  The
// 64 lanes of a wave span (hx, hz), so that one load instruction reads H
// consecutive entries per row; a lane owns TY targets of its class
// consecutive in hy (2 apart in y).  Walking the zone by (dx, dz) columns,
// each parity plane of a column is one run of TY + 2 source rows along hy
// shared by the TY targets (three offsets per target and plane); with
// TY = H the run's rows are the same for the whole wave, so their offsets
// fold into the load instructions.  Columns
// next to the target (|dx|, |dz| <= 1) skip the three dy of the near zone.
// Blocks are dealt to the 8 XCDs so that the 8 frequencies of a chunk, which
// share every 128-byte line of the spectra, run on one XCD back to back.
//
// T = float: the sources and kernel values in FP32 (with TS = float2 the
// level's spectra are stored in FP32 too; the transforms compute in FP64),
// the terms of each (dx, dz) column summed in FP32 and the 36 column sums
// of a target added in FP64.
template <int H, int TY, class T = double, class TS = double2>
__global__ void __launch_bounds__(8 * (H * H * H / TY), sizeof(T) == 4 ? 4 : 8) k_zone_level_y(
    const TS* __restrict__ spec, const typename Vec2<T>::type* __restrict__ khatT, int64_t F,
    int nchunk, TS* __restrict__ out) {
  using T2 = typename Vec2<T>::type;
  constexpr bool kSplit = sizeof(T) == 4;  // FP32 column sums into FP64 totals
  constexpr int n = 2 * H, nn = n * n * n, H3 = H * H * H;
  constexpr int LPC = H3 / TY;   // lanes per class
  constexpr int NT = 8 * LPC;
  static_assert(LPC % 64 == 0, "a class fills whole waves");
  static_assert(H % TY == 0, "whole target runs");
  __shared__ T2 box[nn];
  const int g = blockIdx.x;
  const int chunk = ((g >> 3) >> 3) * 8 + (g & 7);
  if (chunk >= nchunk) return;
  const int k = chunk * 8 + ((g >> 3) & 7);
  const TS* sk = spec + (int64_t)(k >> 3) * nn * 8 + (k & 7);  // node v at sk[8 v]
  // stage: LDS slot i = ((p * H + hx) * H + (hy ^ (hx & 1))) * H + hz,
  // consecutive threads writing consecutive slots.  Flipping the low bit of
  // hy on odd hx puts the two hx of a 16-lane group on different halves of
  // the 64 banks when all lanes read one hy.
  for (int i = threadIdx.x; i < nn; i += NT) {
    const int hz = i % H, hx = (i / (H * H)) % H, hy = ((i / H) % H) ^ (hx & 1), p = i / H3;
    const int x = 2 * hx + (p >> 2), y = 2 * hy + ((p >> 1) & 1), z = 2 * hz + (p & 1);
    const TS v = sk[(int64_t)((x * n + y) * n + z) * 8];
    box[i] = T2{(T)v.x, (T)v.y};
  }
  __syncthreads();
  const int cls = __builtin_amdgcn_readfirstlane(threadIdx.x / LPC);
  const int cx = cls >> 2, cy = (cls >> 1) & 1, cz = cls & 1;
  const int lane = threadIdx.x % LPC;
  const int hz = lane % H, hx = (lane / H) % H, hy0 = (lane / (H * H)) * TY;
  const T2* kf = khatT + (int64_t)k * kKT;
  double re[TY], im[TY];
  T cr[TY], ci[TY];  // the current column's sums (FP32 with kSplit)
#pragma unroll
  for (int t = 0; t < TY; ++t) {
    re[t] = im[t] = 0.0;
    cr[t] = ci[t] = (T)0;
  }
  int fl = 0;  // 1 when the current source column's hx' is odd
  // one parity plane (py) of a column: rows hy0 - 1 + j (j < TY + 2) of the
  // column's (px, pz, hx', hz'); target t reads j = t + m with the kernel of
  // offset dy = 2 m - 2 + py - cy
  auto plane = [&](int col, int kbase, int py, bool m0, bool m1, bool m2) {
    // row hy sits at slot row hy ^ (hx' & 1): one base per parity of hy
    // (32-bit LDS slot offsets, no pointer arithmetic)
    const int pl = col + py * 2 * H3;
    const int pe = pl + fl * H;   // even hy: +H on odd hx'
    const int po = pl - fl * H;   // odd hy: -H on odd hx'
    T2 src[TY + 2];
#pragma unroll
    for (int j = 0; j < TY + 2; ++j) {
      const int hy = (hy0 - 1 + j) & (H - 1);
      src[j] = box[((hy & 1) ? po : pe) + hy * H];
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      if ((m == 0 && !m0) || (m == 1 && !m1) || (m == 2 && !m2)) continue;
      const T2 kd = kf[kbase + 7 * (2 * m - 2 + py - cy + 3)];
      if constexpr (kSplit) {
        // k s = (kx sx - ky sy, kx sy + ky sx) with -ky kept as its own value
        const float kx = vreg(kd.x), ky = vreg(kd.y), nky = vreg(-kd.y);
#pragma unroll
        for (int t = 0; t < TY; ++t) {
          cr[t] = fmaf(kx, src[t + m].x, cr[t]);
          cr[t] = fmaf(nky, src[t + m].y, cr[t]);
          ci[t] = fmaf(kx, src[t + m].y, ci[t]);
          ci[t] = fmaf(ky, src[t + m].x, ci[t]);
        }
      } else {
#pragma unroll
        for (int t = 0; t < TY; ++t) cmac(re[t], im[t], kd, src[t + m]);
      }
    }
  };
  // with kSplit, a finished column's sums go into the FP64 totals
  auto flush = [&]() {
    if constexpr (kSplit) {
#pragma unroll
      for (int t = 0; t < TY; ++t) {
        re[t] += (double)cr[t];
        im[t] += (double)ci[t];
        cr[t] = ci[t] = (T)0;
      }
    }
  };
  for (int sx = -2; sx <= 3; ++sx) {      // source x = 2 hx + cx + dx, sx = cx + dx
    const int dx = sx - cx;
    const int hxs = (hx + (sx >> 1)) & (H - 1);
    fl = hxs & 1;
    const int cxo = (sx & 1) * 4 * H3 + hxs * H * H;
    for (int sz = -2; sz <= 3; ++sz) {
      const int dz = sz - cz;
      const int col = cxo + (sz & 1) * H3 + ((hz + (sz >> 1)) & (H - 1));
      const int kbase = (dx + 3) * 49 + (dz + 3);
      if (abs(dx) > 1 || abs(dz) > 1) {
        plane(col, kbase, 0, true, true, true);
        plane(col, kbase, 1, true, true, true);
      } else if (cy == 0) {  // keep sy = -2, 2 (even) and 3 (odd)
        plane(col, kbase, 0, true, false, true);
        plane(col, kbase, 1, false, false, true);
      } else {               // keep sy = -2 (even), -1 and 3 (odd)
        plane(col, kbase, 0, true, false, false);
        plane(col, kbase, 1, true, false, true);
      }
      flush();
    }
  }
  TS* o = out + (int64_t)(k >> 3) * nn * 8 + (k & 7);
#pragma unroll
  for (int t = 0; t < TY; ++t) {
    const int y = 2 * (hy0 + t) + cy;
    const int v = ((2 * hx + cx) * n + y) * n + (2 * hz + cz);
    o[(int64_t)v * 8] = from_d2<TS>(make_double2(re[t], im[t]));
  }
}

// The 4^3 level (37 offsets periodic, 316 isolated): one wave per frequency,
// lane t the target node t, sources and kernel values in LDS.  The zone:
// periodic, each of the level's nodes once, d_i in [-2, 1]; isolated, d_i in
// [-3, 3] and sources inside the box; always max |d_i| > 1 (Sec. 2).
template <bool ISO>
__global__ void __launch_bounds__(256) k_zone_l2(const double2* __restrict__ spec,
                                                 const double2* __restrict__ khatT,
                                                 double2* __restrict__ out) {
  __shared__ double2 box[4][64];
  __shared__ double2 kk[4][kKT];
  const int w = threadIdx.x >> 6, t = threadIdx.x & 63, k = blockIdx.x * 4 + w;
  box[w][t] = spec[sidx(k, t, 64)];
  for (int i = t; i < kKT; i += 64) kk[w][i] = khatT[(int64_t)k * kKT + i];
  __syncthreads();
  const int tx = t >> 4, ty = (t >> 2) & 3, tz = t & 3;
  constexpr int D0 = ISO ? -3 : -2, D1 = ISO ? 3 : 1;
  double re = 0.0, im = 0.0;
#pragma unroll
  for (int dx = D0; dx <= D1; ++dx)
#pragma unroll
    for (int dy = D0; dy <= D1; ++dy)
#pragma unroll
      for (int dz = D0; dz <= D1; ++dz) {
        if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1) continue;
        const int x = tx + dx, y = ty + dy, z = tz + dz;
        double2 sv = box[w][((x & 3) * 4 + (y & 3)) * 4 + (z & 3)];
        if (ISO && ((unsigned)x > 3u || (unsigned)y > 3u || (unsigned)z > 3u)) sv = make_double2(0.0, 0.0);
        cmac(re, im, kk[w][(dx + 3) * 49 + (dy + 3) * 7 + dz + 3], sv);
      }
  out[sidx(k, t, 64)] = make_double2(re, im);
}

// khatT in FP32.
__global__ void k_khat_f32(const double2* __restrict__ in, int64_t n, float2* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < n) out[i] = make_float2((float)in[i].x, (float)in[i].y);
}

// Kernel spectra of a level, in place in khatT: [x][y][kz] rows of 344 offsets,
// the layout of the finished table.  Along z of K_d[x][y][z] = tab[w(x) - p dx]
// [w(y) - p dy][w(z) - p dz] (tab centred at C), zero on the unused slot p; along
// y, whose results go to their place in the order of k_node_fwd; along x with
// the normalisation.  One thread per offset and column, the column in
// registers, so that every access is a run over the offsets; blockIdx.z takes
// the levels.
//
// In twice FP64's precision, rounded once at the end (`low` holds the low parts
// between the passes, laid out as khatT): the kernel is smooth, so its high
// frequencies are small, but in FP64 they would carry rounding of the size of
// the low ones, which the alternating effective masses of a gridlet amplify.
// Measured on 16^3 cells, two levels, p = 8, against extended precision: relative
// error of the FP64 potential 9.9e-14 with spectra in FP64, 5.2e-14 with these,
// 5.6e-14 by block-Toeplitz products.
//
// Bound: the passes' traffic, 3 writes and 2 reads of twice 12.7 MB a level at p
// = 8, and the sums' own latency: 55 us for two levels (one thread per frequency
// with its twiddles computed for each term and a scattered store, in FP64: 155).
struct KhatLevels {
  const double* tab[16];
  double2 *khat[16], *low[16];
};

// DFT of 2P values in registers, natural order
template <int P, class T>
__device__ __forceinline__ void ddft2(T (&v)[2 * P]) {
  T e[P], o[P];
#pragma unroll
  for (int j = 0; j < P; ++j) {
    e[j] = v[2 * j];
    o[j] = v[2 * j + 1];
  }
  ddft<P, false>(e);
  ddft<P, false>(o);
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const T t = j ? dtwiddle<2 * P, false>(o[j], j) : o[j];
    v[j] = dadd(e[j], t);
    v[j + P] = dsub(e[j], t);
  }
}

__device__ __forceinline__ wide2 load_wide(const double2* h, const double2* l, int64_t i) {
  const double2 a = h[i], b = l[i];
  return {{a.x, b.x}, {a.y, b.y}};
}
__device__ __forceinline__ void store_wide(double2* h, double2* l, int64_t i, wide2 v) {
  h[i] = make_double2(v.x.h, v.y.h);
  l[i] = make_double2(v.x.l, v.y.l);
}

constexpr int kKB = 64;  // offsets per workgroup of the kernel transforms

template <int P>
__global__ void __launch_bounds__(kKB) k_khat_z(KhatLevels lv) {
  constexpr int M = 2 * P, H = P + 1, C = 4 * P - 1, E = 2 * C + 1;
  const int di = blockIdx.y * kKB + threadIdx.x;
  if (di >= kKT) return;
  const int y = blockIdx.x % M, x = blockIdx.x / M;
  wide2 v[M];
#pragma unroll
  for (int z = 0; z < M; ++z) v[z] = wide2{{0.0, 0.0}, {0.0, 0.0}};
  if (x != P && y != P && di < 343) {  // offset 343 is padding
    const int dx = di / 49 - 3, dy = (di / 7) % 7 - 3, dz = di % 7 - 3;
    const int jx = (x < P ? x : x - M) - P * dx, jy = (y < P ? y : y - M) - P * dy;
    const double* row = lv.tab[blockIdx.z] + ((int64_t)(jx + C) * E + (jy + C)) * E + (C - P * dz);
#pragma unroll
    for (int z = 0; z < M; ++z)
      if (z != P) v[z].x.h = row[z < P ? z : z - M];
    ddft2<P>(v);
  }
  const int64_t o = (int64_t)blockIdx.x * H * kKT + di;
#pragma unroll
  for (int k = 0; k < H; ++k) store_wide(lv.khat[blockIdx.z], lv.low[blockIdx.z], o + k * kKT, v[k]);
}

template <int P>
__global__ void __launch_bounds__(kKB) k_khat_y(KhatLevels lv) {
  constexpr int M = 2 * P, H = P + 1;
  const int di = blockIdx.y * kKB + threadIdx.x;
  if (di >= kKT) return;
  const int kz = blockIdx.x % H, x = blockIdx.x / H;
  double2 *h = lv.khat[blockIdx.z], *l = lv.low[blockIdx.z];
  const int64_t c = ((int64_t)x * M * H + kz) * kKT + di;
  wide2 v[M];
#pragma unroll
  for (int y = 0; y < M; ++y) v[y] = load_wide(h, l, c + (int64_t)y * H * kKT);
  ddft2<P>(v);
#pragma unroll
  for (int k = 0; k < M; ++k) store_wide(h, l, c + (int64_t)((k & 1) * P + (k >> 1)) * H * kKT, v[k]);
}

template <int P>
__global__ void __launch_bounds__(kKB) k_khat_x(KhatLevels lv) {
  constexpr int M = 2 * P, H = P + 1;
  constexpr double scale = 1.0 / (M * M * M);
  const int di = blockIdx.y * kKB + threadIdx.x;
  if (di >= kKT) return;
  double2 *h = lv.khat[blockIdx.z], *l = lv.low[blockIdx.z];
  const int64_t c = (int64_t)blockIdx.x * kKT + di;  // row y' H + kz
  wide2 v[M];
#pragma unroll
  for (int x = 0; x < M; ++x) v[x] = load_wide(h, l, c + (int64_t)x * M * H * kKT);
  ddft2<P>(v);
#pragma unroll
  for (int k = 0; k < M; ++k)
    h[c + (int64_t)k * M * H * kKT] = make_double2(v[k].x.h * scale, v[k].y.h * scale);
}

template <int P>
hipError_t khat_levels(const M2LSpectral* f, const std::vector<double*>& tab64, hipStream_t st) {
  constexpr int M = 2 * P, H = P + 1, nb = (kKT + kKB - 1) / kKB;
  KhatLevels lv{};
  for (int l = 2; l <= f->L; ++l) {
    lv.tab[l - 2] = tab64[l];
    lv.khat[l - 2] = f->khatT[l];
    lv.low[l - 2] = f->out + (l - 2) * f->F * kKT;  // before any spectra
  }
  const unsigned nl = f->L - 1;
  k_khat_z<P><<<dim3(M * M, nb, nl), kKB, 0, st>>>(lv);
  k_khat_y<P><<<dim3(M * H, nb, nl), kKB, 0, st>>>(lv);
  k_khat_x<P><<<dim3(M * H, nb, nl), kKB, 0, st>>>(lv);
  return hipGetLastError();
}

inline hipError_t tbegin(KernelTimer* kt, hipStream_t st) { return kt ? kt->begin(st) : hipSuccess; }
inline hipError_t tend(KernelTimer* kt, hipStream_t st, int part, hipError_t e) {
  if (e != hipSuccess || !kt) return e;
  return kt->end(st, part);
}

template <int HX, int HY, int HZ, int G, bool WRAP>
void zone_oct_as(const M2LSpectral* f, int l, int n, int isolated, int nchunk, hipStream_t st) {
  const int hn = n / 2, tiles = (hn / HX) * (hn / HY) * (hn / HZ);
  // the chunks rounded up to a multiple of 8, times their frequencies, per tile
  const unsigned grid = (unsigned)((nchunk + 7) / 8 * 8 * kFC) * (unsigned)tiles;
  k_zone_oct<HX, HY, HZ, G, WRAP><<<grid, HX * HY * HZ * 4 / G, 0, st>>>(f->spec[l], f->khatT[l], n,
                                                                         isolated, nchunk, f->out);
}

// The octet products of a level of n >= 8 nodes per axis: the periodic 8^3
// level is one tile; other levels take tiles of 4 x 4 x 8 parents (4^3 on the
// isolated 8^3 level) with a halo (46 KiB, three tiles per CU: while one
// stages its sources another multiplies).
void zone_oct(const M2LSpectral* f, int l, int n, int isolated, int nchunk, hipStream_t st) {
  if (n == 8 && !isolated)
    zone_oct_as<4, 4, 4, 1, true>(f, l, n, isolated, nchunk, st);
  else if (n == 8)
    zone_oct_as<4, 4, 4, 1, false>(f, l, n, isolated, nchunk, st);
  else
    zone_oct_as<4, 4, 8, 2, false>(f, l, n, isolated, nchunk, st);
}

// The zone sums of a level from its spectra (FP64) into f->out.
void zone_sums(const M2LSpectral* f, int l, int isolated, hipStream_t st) {
  const int n = 1 << l;
  const int nchunk = (int)(f->F / kFC);
  if (n == 16 && !isolated) {  // the whole level per frequency, eight targets per lane
    const unsigned cgrid = (unsigned)((nchunk + 7) / 8 * 64);  // chunks rounded up to 8, times 8
    k_zone_level_y<8, 8><<<cgrid, 512, 0, st>>>(f->spec[l], f->khatT[l], f->F, nchunk, f->out);
  } else if (n == 4) {
    if (isolated)
      k_zone_l2<true><<<(unsigned)(f->F / 4), 256, 0, st>>>(f->spec[l], f->khatT[l], f->out);
    else
      k_zone_l2<false><<<(unsigned)(f->F / 4), 256, 0, st>>>(f->spec[l], f->khatT[l], f->out);
  } else {
    zone_oct(f, l, n, isolated, nchunk, st);
  }
}

template <int P>
hipError_t run_level(const M2LSpectral* f, int l, const void* Ml, int m64, void* Pl, int p64,
                     int accumulate, int isolated, int cols32, hipStream_t st, KernelTimer* kt) {
  const int n = 1 << l;
  const int64_t nn = (int64_t)n * n * n;
  constexpr int NT = node_threads<P>();
  // the 16^3 leaf level in FP32 columns: its spectra stored as float2
  const bool f32 = n == 16 && !isolated && cols32 && f->f32 && l == f->L;
  float2* spec32 = reinterpret_cast<float2*>(f->spec[l]);
  float2* out32 = reinterpret_cast<float2*>(f->out);
  hipError_t e = tbegin(kt, st);
  if (e != hipSuccess) return e;
  if (m64 && f32)
    k_node_fwd<P, double, float2><<<(unsigned)nn, NT, 0, st>>>((const double*)Ml, nn, spec32);
  else if (f32)
    k_node_fwd<P, float, float2><<<(unsigned)nn, NT, 0, st>>>((const float*)Ml, nn, spec32);
  else if (m64)
    k_node_fwd<P, double><<<(unsigned)nn, NT, 0, st>>>((const double*)Ml, nn, f->spec[l]);
  else
    k_node_fwd<P, float><<<(unsigned)nn, NT, 0, st>>>((const float*)Ml, nn, f->spec[l]);
  e = tend(kt, st, 0, hipGetLastError());
  if (e == hipSuccess) e = tbegin(kt, st);
  if (e != hipSuccess) return e;
  if (f32)  // FP32 columns
    k_zone_level_y<8, 8, float, float2><<<(unsigned)((f->F / kFC + 7) / 8 * 64), 512, 0, st>>>(
        spec32, f->khatT32, f->F, (int)(f->F / kFC), out32);
  else
    zone_sums(f, l, isolated, st);
  e = tend(kt, st, 1, hipGetLastError());
  if (e == hipSuccess) e = tbegin(kt, st);
  if (e != hipSuccess) return e;
  if (p64 && f32)
    k_node_inv<P, double, float2><<<(unsigned)nn, NT, 0, st>>>(out32, nn, accumulate, (double*)Pl);
  else if (f32)
    k_node_inv<P, float, float2><<<(unsigned)nn, NT, 0, st>>>(out32, nn, accumulate, (float*)Pl);
  else if (p64)
    k_node_inv<P, double><<<(unsigned)nn, NT, 0, st>>>(f->out, nn, accumulate, (double*)Pl);
  else
    k_node_inv<P, float><<<(unsigned)nn, NT, 0, st>>>(f->out, nn, accumulate, (float*)Pl);
  return tend(kt, st, 2, hipGetLastError());
}

}  // namespace

void m2l_spectral_destroy(M2LSpectral* f) {
  if (!f) return;
  (void)hipFree(f->mem);
  delete f;
}

namespace {
// Values per frequency of the node spectra (every level's, and the sums of the
// largest), which also hold the low parts of every level's kernels while these
// are transformed
size_t spectra_per_freq(int L) {
  size_t n = (size_t)1 << (3 * L);
  for (int l = 2; l <= L; ++l) n += (size_t)1 << (3 * l);
  return std::max(n, (size_t)(L - 1) * kKT);
}
}  // namespace

size_t m2l_spectral_bytes(int L, int p) {
  const size_t F = (size_t)(2 * p) * (2 * p) * (p + 1);
  return F * ((spectra_per_freq(L) + (size_t)(L - 1) * kKT) * sizeof(double2) +
              (L == 4 ? kKT * sizeof(float2) : 0));
}

int m2l_spectral_levels(const M2LSpectral* f) { return f->L; }

hipError_t m2l_spectral_create(int L, int p, M2LSpectral** out) {
  *out = nullptr;
  if (p < 1 || p > 10 || L < 2) return hipErrorInvalidValue;
  void* mem = nullptr;
  const hipError_t e = hipMalloc(&mem, m2l_spectral_bytes(L, p));
  if (e != hipSuccess) return e;
  M2LSpectral* f = new M2LSpectral;
  f->L = L;
  f->p = p;
  f->F = (int64_t)(2 * p) * (2 * p) * (p + 1);
  f->mem = mem;
  double2* at = static_cast<double2*>(mem);
  auto take = [&](int64_t n) {
    double2* a = at;
    at += n;
    return a;
  };
  f->out = take(f->F * (int64_t)spectra_per_freq(L));
  f->spec.assign(L + 1, nullptr);
  double2* sp = f->out + (f->F << (3 * L));
  for (int l = L; l >= 2; --l) {
    f->spec[l] = sp;
    sp += f->F << (3 * l);
  }
  f->khatT.assign(L + 1, nullptr);
  for (int l = 2; l <= L; ++l) f->khatT[l] = take(f->F * kKT);
  if (L == 4) f->khatT32 = reinterpret_cast<float2*>(at);
  *out = f;
  return hipSuccess;
}

namespace {
hipError_t khat_f32(const M2LSpectral* f, hipStream_t st) {
  k_khat_f32<<<nblk(f->F * kKT), kThreads, 0, st>>>(f->khatT[f->L], f->F * kKT, f->khatT32);
  return hipGetLastError();
}
}  // namespace

hipError_t m2l_spectral_keep_f32(M2LSpectral* f, hipStream_t st) {
  if (f->f32 || !f->khatT32) return hipSuccess;
  hipError_t e = khat_f32(f, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  f->f32 = e == hipSuccess;
  return e;
}

hipError_t m2l_spectral_tables(M2LSpectral* f, const std::vector<double*>& tab64, hipStream_t st) {
  hipError_t e = with_p<1, 10>(f->p, [&](auto P) { return khat_levels<decltype(P)::value>(f, tab64, st); });
  if (e == hipSuccess && f->f32) e = khat_f32(f, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  return e;
}

hipError_t m2l_spectral_level(const M2LSpectral* f, int l, const void* Ml, int m64, void* Pl, int p64,
                              int accumulate, int isolated, int cols32, hipStream_t st,
                              KernelTimer* kt) {
  if (l < 2 || l > f->L) return hipErrorInvalidValue;
  return with_p<1, 10>(f->p, [&](auto P) {
    return run_level<decltype(P)::value>(f, l, Ml, m64, Pl, p64, accumulate, isolated, cols32, st, kt);
  });
}

hipError_t m2l_spectral_sums(const M2LSpectral* f, int l, int isolated, hipStream_t st) {
  if (l < 2 || l > f->L) return hipErrorInvalidValue;
  zone_sums(f, l, isolated, st);
  return hipGetLastError();
}

}  // namespace pfmm
