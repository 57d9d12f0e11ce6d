// Learned correction of the interaction-zone Green's-function tables.
//
// The paper defines an "optimal" Green's function G_* as the one with which
// the FMM reproduces the PM solution (Sec. 3, Eq. 8), approximates it by the
// closed form G_S1 (Eq. 9), and suggests parameterising G_* by many values
// and minimising the FMM-vs-PM error (Sec. 4).  Here a small MLP
// f_theta(|j| sorted / (4p), (|j| sorted mod p) / p, level / 8, p / 10) of the
// table offset j = a - a' - p d (its cube invariants and in-gridlet residues),
// the level and p gives every table entry
// T_l[j] = G(eta_l j) (1 + delta), delta = kappa f_theta with the fixed output
// scale kappa = 1e-4 (the corrections that matter are of the size of the
// FMM-vs-PM residual), of the interaction-zone convolution (Eq. 6); the near
// zone keeps G.  The network is invariant under the 48
// symmetries of the cube, so the corrected operator keeps the FMM symmetric.
// An untrained network (zero output layer) is exactly the uncorrected G.
//
// Training minimises the mean-removed relative residual
//     loss = sum_i r_i^2 / sum_i (phi_t,i - mean)^2,   r = phi - phi_t - mean(phi - phi_t)
// The FMM potential is linear in every table, so
//     d loss / d T_l[j] = sum_t sum_{d in IZ(t)} sum_{a - a' - p d = j} lambda_l[t][a] M_l[t+d][a']
// with the adjoint lambda_l = (M2M)^(L-l) P2M(2 r / norm): the transposes of
// L2L (Eq. 7) and L2P.  The kernels below compute the residual, the table
// gradient, its pull-back to the network output, the network's gradient, and
// Adam; the forward solve and the adjoint sweep reuse the solve's kernels.
#include "internal.h"

#include <cstdint>

namespace pfmm {
namespace {

constexpr int kH = 64;           // hidden width
constexpr float kKappa = 1e-4f;  // output scale: delta = kappa * network output

__device__ inline float silu(float z) { return z / (1.f + expf(-z)); }
__device__ inline float dsilu(float z) {
  const float s = 1.f / (1.f + expf(-z));
  return s * (1.f + z * (1.f - s));
}
__device__ inline float rb(float x, int bf16) { return bf16 ? (float)(__bf16)x : x; }

// theta layout: W1[64][kMlpIn] b1[64] W2[64][64] b2[64] W3[64] b3
constexpr int oW1 = 0, oB1 = kH * kMlpIn, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH,
              oB3 = oW3 + kH;
static_assert(oB3 + 1 == kMlpParams, "network layout");

// The network kernels take 64 hidden units x 4 groups of entries a block: a
// thread is one unit, its weights in registers, the activations of the entries
// in LDS (one address a wave).  One thread per entry left 26 blocks of a wave
// for the 1632 entries of p = 4, L = 3 (forward 50 us, backward 93 us).
constexpr int kFwdEntries = 16, kBwdEntries = 32;

// Network output for every entry; with bf16 = 1 the weights, inputs and
// activations are rounded to bf16 before each product (FP32 accumulation).
__global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ theta,
                                                     const float* __restrict__ feats, int n, int bf16,
                                                     float* __restrict__ delta) {
  constexpr int EB = kFwdEntries, EG = EB / 4;
  __shared__ float X[EB][kMlpIn], H1[EB][kH], H2[EB][kH + 1];
  const int i = threadIdx.x & 63, grp = threadIdx.x >> 6, e0 = blockIdx.x * EB;
  float w1[kMlpIn], w2[kH];
#pragma unroll
  for (int k = 0; k < kMlpIn; ++k) w1[k] = rb(theta[oW1 + i * kMlpIn + k], bf16);
#pragma unroll
  for (int k = 0; k < kH; ++k) w2[k] = rb(theta[oW2 + i * kH + k], bf16);
  const float b1 = rb(theta[oB1 + i], bf16), b2 = rb(theta[oB2 + i], bf16);
  if (threadIdx.x < EB * kMlpIn) {
    const int e = e0 + threadIdx.x / kMlpIn;
    X[threadIdx.x / kMlpIn][threadIdx.x % kMlpIn] =
        e < n ? rb(feats[e * kMlpIn + threadIdx.x % kMlpIn], bf16) : 0.f;
  }
  __syncthreads();
  for (int u = 0; u < EG; ++u) {
    const int e = grp * EG + u;
    float z = b1;
#pragma unroll
    for (int k = 0; k < kMlpIn; ++k) z += w1[k] * X[e][k];
    H1[e][i] = rb(silu(z), bf16);
  }
  __syncthreads();
  for (int u = 0; u < EG; ++u) {
    const int e = grp * EG + u;
    float z = b2;
#pragma unroll
    for (int k = 0; k < kH; ++k) z += w2[k] * H1[e][k];
    H2[e][i] = rb(silu(z), bf16);
  }
  __syncthreads();
  if (threadIdx.x < EB && e0 + (int)threadIdx.x < n) {
    float out = rb(theta[oB3], bf16);
    for (int k = 0; k < kH; ++k) out += rb(theta[oW3 + k], bf16) * H2[threadIdx.x][k];
    delta[e0 + threadIdx.x] = kKappa * out;
  }
}

// T[j] = G0[j] (1 + delta[uidx[j]]) in FP64 and, unless t32 is null, FP32
__global__ void k_apply_correction(const double* __restrict__ g0, const float* __restrict__ delta,
                                   const int* __restrict__ uidx, int64_t n,
                                   double* __restrict__ t64, float* __restrict__ t32) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double v = g0[i] * (1.0 + (double)delta[uidx[i]]);
  t64[i] = v;
  if (t32) t32[i] = (float)v;
}

// Partial sums over the mesh of d = phi - t, d^2, t, t^2 (FP64), one block each.
__global__ void k_resid_partial(const float* __restrict__ phi, const float* __restrict__ t,
                                int64_t n, double* __restrict__ part) {
  __shared__ double sd[256], sdd[256], st[256], stt[256];
  double a = 0, b = 0, c = 0, e = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double d = (double)phi[i] - (double)t[i], tv = t[i];
    a += d;
    b += d * d;
    c += tv;
    e += tv * tv;
  }
  sd[threadIdx.x] = a;
  sdd[threadIdx.x] = b;
  st[threadIdx.x] = c;
  stt[threadIdx.x] = e;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      sd[threadIdx.x] += sd[threadIdx.x + s];
      sdd[threadIdx.x] += sdd[threadIdx.x + s];
      st[threadIdx.x] += st[threadIdx.x + s];
      stt[threadIdx.x] += stt[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[blockIdx.x * 4 + 0] = sd[0];
    part[blockIdx.x * 4 + 1] = sdd[0];
    part[blockIdx.x * 4 + 2] = st[0];
    part[blockIdx.x * 4 + 3] = stt[0];
  }
}

// out[0] = mean d, out[1] = loss, out[2] = norm, out[3] = mean t: the 1024 block
// partials summed by a tree in one block of 1024 threads (one thread walking
// them in order took 137 us, all latency)
__global__ __launch_bounds__(1024) void k_resid_final(const double* __restrict__ part, int64_t n,
                                                      double* __restrict__ out) {
  __shared__ double sh[4][1024];
  const int tid = threadIdx.x;
  for (int c = 0; c < 4; ++c) sh[c][tid] = part[tid * 4 + c];
  __syncthreads();
  for (int h = 512; h > 0; h >>= 1) {
    if (tid < h)
      for (int c = 0; c < 4; ++c) sh[c][tid] += sh[c][tid + h];
    __syncthreads();
  }
  if (tid) return;
  const double a = sh[0][0], b = sh[1][0], c = sh[2][0], e = sh[3][0];
  const double md = a / (double)n, mt = c / (double)n;
  const double norm = e - (double)n * mt * mt;
  out[0] = md;
  out[1] = (b - (double)n * md * md) / norm;
  out[2] = norm;
  out[3] = mt;
}

// r = 2 (phi - t - mean) / norm  (d loss / d phi)
__global__ void k_resid_scale(const float* __restrict__ phi, const float* __restrict__ t,
                              const double* __restrict__ stats, int64_t n, float* __restrict__ r) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  r[i] = (float)(2.0 * ((double)phi[i] - (double)t[i] - stats[0]) / stats[2]);
}

// Table gradient, one block per (class, offset, split of the class's targets):
// window entries w of the (2q-1)^3 slice around -q d get the sum over targets t
// and points a of lambda[t][a] M[t+d][a - w'] (w' = w - (q-1) per axis), in FP64.
// A thread owns the 2q - 1 entries of one (w_x, w_y) and walks the row pairs
// (a_x, a_y): two rows of q values from LDS feed q^2 multiply-adds in registers.
// G groups of threads take targets in turn; their sums are added in order.
// MESH: lambda and M are meshes [n q]^3 (the near zone's table), else [node][q^3].
// (One thread per entry with both factors of every product read from LDS, and a
// gather that walked every offset, took 340 + 200 us at p = 4 on the 8^3 level
// where this takes 84 + 18.  G_*'s near table, one block per entry walking
// the whole mesh, 5.1 ms at 64^3, s = 4, now 0.14.)  The row pairs of a lane number
// (q - |w_x|)(q - |w_y|), a third of the largest on average: that is the bound.
template <int Q>
struct GradShape {
  static constexpr int S = 2 * Q - 1, P = S * S, Q3 = Q * Q * Q;
  static constexpr int NT = P > 256 ? 384 : 256, G = NT / P;   // threads, groups
  static constexpr int TB = G >= 4 ? G : Q >= 9 ? 2 : Q == 5 || Q == 6 ? 2 * G : 4;  // targets staged
};

template <int Q, class T, bool MESH>
__global__ __launch_bounds__(GradShape<Q>::NT) void k_table_grad(int n, int m, int noff, int splits,
                                                                 const int* __restrict__ offs,
                                                                 const T* __restrict__ lam,
                                                                 const T* __restrict__ M,
                                                                 double* __restrict__ part) {
  using Sh = GradShape<Q>;
  constexpr int S = Sh::S, P = Sh::P, Q3 = Sh::Q3, NT = Sh::NT, G = Sh::G, TB = Sh::TB;
  constexpr size_t kStage = 2 * TB * Q3 * sizeof(T), kRed = G > 1 ? (size_t)G * P * S * sizeof(double) : 0;
  __shared__ __align__(16) unsigned char smraw[kStage > kRed ? kStage : kRed];
  T* sl = reinterpret_cast<T*>(smraw);  // lambda of the staged targets
  T* sm = sl + TB * Q3;                 // M of their sources
  const int sp = blockIdx.x % splits, ck = blockIdx.x / splits;
  const int cls = ck / noff;
  const int pk = offs[ck];
  const int dx = ((pk >> 16) & 255) - 128, dy = ((pk >> 8) & 255) - 128, dz = (pk & 255) - 128;
  const int cx = cls / (m * m), cy = (cls / m) % m, cz = cls % m;
  const int nk = n / m, ntarg = nk * nk * nk;
  const int tb = (int)((int64_t)ntarg * sp / splits), te = (int)((int64_t)ntarg * (sp + 1) / splits);
  const int grp = threadIdx.x / P, pr = threadIdx.x % P;
  const int wx = pr / S - (Q - 1), wy = pr % S - (Q - 1);
  auto at = [&](int x, int y, int z, int e) -> size_t {  // value e of block (x, y, z)
    if (!MESH) return (((size_t)x * n + y) * n + z) * Q3 + e;
    const size_t N = (size_t)n * Q;
    return ((size_t)(x * Q + e / (Q * Q)) * N + (y * Q + (e / Q) % Q)) * N + (z * Q + e % Q);
  };
  double acc[S];
#pragma unroll
  for (int j = 0; j < S; ++j) acc[j] = 0.0;
  for (int t0 = tb; t0 < te; t0 += TB) {
    const int cnt = te - t0 < TB ? te - t0 : TB;
    __syncthreads();
    for (int i = threadIdx.x; i < cnt * Q3; i += NT) {
      const int t = t0 + i / Q3, e = i % Q3;
      const int tx = cx + m * (t / (nk * nk)), ty = cy + m * ((t / nk) % nk), tz = cz + m * (t % nk);
      sl[i] = lam[at(tx, ty, tz, e)];
      sm[i] = M[at((tx + dx) & (n - 1), (ty + dy) & (n - 1), (tz + dz) & (n - 1), e)];
    }
    __syncthreads();
    if (grp < G) {
      for (int tl = grp; tl < cnt; tl += G) {
        for (int ax = wx > 0 ? wx : 0; ax < (wx < 0 ? Q + wx : Q); ++ax)
          for (int ay = wy > 0 ? wy : 0; ay < (wy < 0 ? Q + wy : Q); ++ay) {
            const T* lr = sl + tl * Q3 + (ax * Q + ay) * Q;
            const T* mr = sm + tl * Q3 + ((ax - wx) * Q + ay - wy) * Q;
            double lv[Q], mv[Q];
#pragma unroll
            for (int j = 0; j < Q; ++j) {
              lv[j] = (double)lr[j];
              mv[j] = (double)mr[j];
            }
#pragma unroll
            for (int az = 0; az < Q; ++az)
#pragma unroll
              for (int bz = 0; bz < Q; ++bz)
                acc[az - bz + Q - 1] = fma(lv[az], mv[bz], acc[az - bz + Q - 1]);
          }
      }
    }
  }
  double* o = part + (size_t)blockIdx.x * (P * S);
  if constexpr (G == 1) {
    if (grp == 0)
#pragma unroll
      for (int j = 0; j < S; ++j) o[pr * S + j] = acc[j];
  } else {
    double* red = reinterpret_cast<double*>(smraw);  // [group][w]
    __syncthreads();
    if (grp < G)
#pragma unroll
      for (int j = 0; j < S; ++j) red[(grp * P + pr) * S + j] = acc[j];
    __syncthreads();
    for (int w = threadIdx.x; w < P * S; w += NT) {
      double v = 0.0;
      for (int g = 0; g < G; ++g) v += red[g * P * S + w];
      o[w] = v;
    }
  }
}

// g[j] = scale times the sum over the (class, offset, split) windows holding j:
// per axis at most two offsets d have |j + q d| <= q - 1.  Table extent E = 2C+1;
// `where` finds an offset of [-3, 3]^3 in a class's list.  Eight lanes share an
// entry (each takes every eighth (class, split), in order, then a tree), so its
// loads are in flight together.
__global__ __launch_bounds__(256) void k_table_grad_gather(const double* __restrict__ part, int m3, int noff,
                                                           int splits, const int* __restrict__ offs, int q,
                                                           int C, double scale, double* __restrict__ g) {
  __shared__ short where[8 * 343];
  for (int i = threadIdx.x; i < m3 * 343; i += 256) where[i] = -1;
  __syncthreads();
  for (int i = threadIdx.x; i < m3 * noff; i += 256) {
    const int pk = offs[i];
    const int dx = ((pk >> 16) & 255) - 128, dy = ((pk >> 8) & 255) - 128, dz = (pk & 255) - 128;
    where[i / noff * 343 + (dx + 3) * 49 + (dy + 3) * 7 + dz + 3] = (short)(i % noff);
  }
  __syncthreads();
  const int E = 2 * C + 1;
  const int64_t i = (int64_t)blockIdx.x * 32 + (threadIdx.x >> 3);
  if (i >= (int64_t)E * E * E) return;
  const int l8 = threadIdx.x & 7;
  const int j[3] = {(int)(i / ((int64_t)E * E)) - C, (int)((i / E) % E) - C, (int)(i % E) - C};
  const int S = 2 * q - 1, nw = S * S * S;
  int lo[3], hi[3];  // offsets with -(q - 1) <= j + q d <= q - 1
  for (int a = 0; a < 3; ++a) {
    const int d = (8 * q - j[a]) / q - 8;  // floor(-j / q), |j| < 4q: j + q d in (-q, 0]
    lo[a] = d < -3 ? -3 : d;
    hi[a] = j[a] + q * d < 0 && d < 3 ? d + 1 : d;
  }
  double s = 0.0;
  for (int dx = lo[0]; dx <= hi[0]; ++dx)
    for (int dy = lo[1]; dy <= hi[1]; ++dy)
      for (int dz = lo[2]; dz <= hi[2]; ++dz) {
        const int w = ((j[0] + q * dx + q - 1) * S + (j[1] + q * dy + q - 1)) * S + (j[2] + q * dz + q - 1);
        const int d = (dx + 3) * 49 + (dy + 3) * 7 + dz + 3;
        for (int cr = l8; cr < m3 * splits; cr += 8) {
          const int c = cr / splits, k = where[c * 343 + d];
          if (k >= 0) s += part[(((size_t)c * noff + k) * splits + cr % splits) * nw + w];
        }
      }
#pragma unroll
  for (int h = 4; h > 0; h >>= 1) s += __shfl_down(s, h, 8);
  if (l8 == 0) g[i] = scale * s;
}

// d loss / d delta[u] += sum_{j in orbit(u)} g[j] G0[j]
// (one wave per orbit, its up to 48 scattered entries at once, summed by a tree)
__global__ __launch_bounds__(256) void k_orbit_gather(const double* __restrict__ g,
                                                      const double* __restrict__ g0,
                                                      const int* __restrict__ ptr,
                                                      const int* __restrict__ pos, int nu,
                                                      float* __restrict__ ddelta) {
  const int u = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (u >= nu) return;
  double s = 0.0;
  for (int k = ptr[u] + lane; k < ptr[u + 1]; k += 64) s += g[pos[k]] * g0[pos[k]];
#pragma unroll
  for (int h = 32; h > 0; h >>= 1) s += __shfl_down(s, h);
  if (lane == 0) ddelta[u] += (float)s;
}

// Network gradient for kBwdEntries entries per block (FP32), written as one
// partial gradient per block; every gradient component is summed by one thread
// in entry order.
__global__ __launch_bounds__(256) void k_mlp_backward(const float* __restrict__ theta,
                                                      const float* __restrict__ feats,
                                                      const float* __restrict__ ddelta, int n,
                                                      float* __restrict__ part) {
  constexpr int EB = kBwdEntries, EG = EB / 4;
  __shared__ float X[EB][kMlpIn], DD[EB];
  __shared__ float H1[EB][kH], H2[EB][kH], DZ2[EB][kH], DZ1[EB][kH];
  const int i = threadIdx.x & 63, grp = threadIdx.x >> 6, e0 = blockIdx.x * EB;
  float w1[kMlpIn], w2[kH];  // the unit's rows
#pragma unroll
  for (int k = 0; k < kMlpIn; ++k) w1[k] = theta[oW1 + i * kMlpIn + k];
#pragma unroll
  for (int k = 0; k < kH; ++k) w2[k] = theta[oW2 + i * kH + k];
  const float b1 = theta[oB1 + i], b2 = theta[oB2 + i], w3 = theta[oW3 + i];
  {
    const int e = e0 + threadIdx.x / kMlpIn;
    X[threadIdx.x / kMlpIn][threadIdx.x % kMlpIn] = e < n ? feats[e * kMlpIn + threadIdx.x % kMlpIn] : 0.f;
    static_assert(EB * kMlpIn == 256, "one input a thread");
    if (threadIdx.x < EB)  // d loss / d (network output)
      DD[threadIdx.x] = e0 + (int)threadIdx.x < n ? kKappa * ddelta[e0 + threadIdx.x] : 0.f;
  }
  __syncthreads();
  float z1[EG];
#pragma unroll
  for (int u = 0; u < EG; ++u) {
    const int e = grp * EG + u;
    float z = b1;
#pragma unroll
    for (int k = 0; k < kMlpIn; ++k) z += w1[k] * X[e][k];
    z1[u] = z;
    H1[e][i] = silu(z);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < EG; ++u) {
    const int e = grp * EG + u;
    float z = b2;
#pragma unroll
    for (int k = 0; k < kH; ++k) z += w2[k] * H1[e][k];
    H2[e][i] = silu(z);
    DZ2[e][i] = DD[e] * w3 * dsilu(z);
  }
#pragma unroll
  for (int k = 0; k < kH; ++k) w2[k] = theta[oW2 + k * kH + i];  // now the unit's column
  __syncthreads();
#pragma unroll
  for (int u = 0; u < EG; ++u) {
    const int e = grp * EG + u;
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < kH; ++k) v += w2[k] * DZ2[e][k];
    DZ1[e][i] = v * dsilu(z1[u]);
  }
  __syncthreads();
  float* out = part + (size_t)blockIdx.x * kMlpParams;
  for (int r0 = grp * 16; r0 < grp * 16 + 16; ++r0) {  // rows r0 of W2, column i
    float v = 0.f;
#pragma unroll 8
    for (int e = 0; e < EB; ++e) v += DZ2[e][r0] * H1[e][i];
    out[oW2 + r0 * kH + i] = v;
  }
  for (int k = grp * 2; k < grp * 2 + 2; ++k) {
    float v = 0.f;
    for (int e = 0; e < EB; ++e) v += DZ1[e][i] * X[e][k];
    out[oW1 + i * kMlpIn + k] = v;
  }
  float v = 0.f;
  if (grp == 0) {
    for (int e = 0; e < EB; ++e) v += DZ1[e][i];
    out[oB1 + i] = v;
  } else if (grp == 1) {
    for (int e = 0; e < EB; ++e) v += DZ2[e][i];
    out[oB2 + i] = v;
  } else if (grp == 2) {
    for (int e = 0; e < EB; ++e) v += DD[e] * H2[e][i];
    out[oW3 + i] = v;
  } else if (i == 0) {
    for (int e = 0; e < EB; ++e) v += DD[e];
    out[oB3] = v;
  }
}

// g += the blocks' partial gradients, in order, summed in FP64
__global__ void k_sum_partials(const float* __restrict__ part, int nblk, float* __restrict__ g) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kMlpParams) return;
  double s = 0.0;
#pragma unroll 8
  for (int b = 0; b < nblk; ++b) s += (double)part[(size_t)b * kMlpParams + i];
  g[i] += (float)s;
}

// Adam (Kingma & Ba) on the averaged gradient g / count over n parameters;
// clears g.
__global__ void k_adam(float* __restrict__ th, float* __restrict__ m1, float* __restrict__ m2,
                       float* __restrict__ g, int n, float count, float lr, float b1, float b2,
                       float eps, int step) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i] / count;
  m1[i] = b1 * m1[i] + (1.f - b1) * gi;
  m2[i] = b2 * m2[i] + (1.f - b2) * gi * gi;
  const float mh = m1[i] / (1.f - powf(b1, (float)step));
  const float vh = m2[i] / (1.f - powf(b2, (float)step));
  th[i] -= lr * mh / (sqrtf(vh) + eps);
  g[i] = 0.f;
}

__global__ void k_add_into(float* __restrict__ dst, const float* __restrict__ src, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] += src[i];
}

inline unsigned nb(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t mlp_forward(const float* theta, const float* feats, int n, int bf16, float* delta,
                       hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_forward, dim3(nb(n, kFwdEntries)), dim3(256), 0, st, theta, feats, n, bf16, delta);
  return hipGetLastError();
}

hipError_t apply_correction(const double* g0, const float* delta, const int* uidx, int64_t n,
                            double* t64, float* t32, hipStream_t st) {
  hipLaunchKernelGGL(k_apply_correction, dim3(nb(n, 256)), dim3(256), 0, st, g0, delta, uidx, n,
                     t64, t32);
  return hipGetLastError();
}

hipError_t residual(const float* phi, const float* t, int64_t n, double* part, double* stats,
                    float* r, hipStream_t st) {
  constexpr int nblk = 1024;  // k_resid_final sums one partial a thread
  hipLaunchKernelGGL(k_resid_partial, dim3(nblk), dim3(256), 0, st, phi, t, n, part);
  hipLaunchKernelGGL(k_resid_final, dim3(1), dim3(nblk), 0, st, part, n, stats);
  hipLaunchKernelGGL(k_resid_scale, dim3(nb(n, 256)), dim3(256), 0, st, phi, t, stats, n, r);
  return hipGetLastError();
}

namespace {
// Parts each class's targets are split into: at least 1024 blocks.
int grad_splits(int n, int m, int noff) {
  const int m3 = m * m * m, nk = n / m;
  const int want = (1024 + m3 * noff - 1) / (m3 * noff);
  return want < nk * nk * nk ? want : nk * nk * nk;
}

template <int Q, bool MESH>
void launch_grad(int n, int m, int noff, int splits, const int* offs, const void* lam, const void* M,
                 int fp64, double* part, hipStream_t st) {
  const dim3 grid(m * m * m * noff * splits), block(GradShape<Q>::NT);
  if (!MESH && fp64)
    k_table_grad<Q, double, false><<<grid, block, 0, st>>>(n, m, noff, splits, offs, (const double*)lam,
                                                          (const double*)M, part);
  else
    k_table_grad<Q, float, MESH><<<grid, block, 0, st>>>(n, m, noff, splits, offs, (const float*)lam,
                                                        (const float*)M, part);
}

template <bool MESH>
hipError_t grad(int n, int m, int q, int noff, const int* offs, const void* lam, const void* M, int fp64,
                int C, double scale, double* part, double* g, hipStream_t st) {
  const int sp = grad_splits(n, m, noff), m3 = m * m * m;
  switch (q) {
    case 1: launch_grad<1, MESH>(n, m, noff, sp, offs, lam, M, fp64, part, st); break;
    case 2: launch_grad<2, MESH>(n, m, noff, sp, offs, lam, M, fp64, part, st); break;
    case 3: launch_grad<3, MESH>(n, m, noff, sp, offs, lam, M, fp64, part, st); break;
    case 4: launch_grad<4, MESH>(n, m, noff, sp, offs, lam, M, fp64, part, st); break;
    case 5: launch_grad<5, MESH>(n, m, noff, sp, offs, lam, M, fp64, part, st); break;
    case 6: launch_grad<6, MESH>(n, m, noff, sp, offs, lam, M, fp64, part, st); break;
    case 7: launch_grad<7, MESH>(n, m, noff, sp, offs, lam, M, fp64, part, st); break;
    case 8: launch_grad<8, MESH>(n, m, noff, sp, offs, lam, M, fp64, part, st); break;
    case 9: launch_grad<9, MESH>(n, m, noff, sp, offs, lam, M, fp64, part, st); break;
    case 10: launch_grad<10, MESH>(n, m, noff, sp, offs, lam, M, fp64, part, st); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t E = 2 * C + 1;
  hipLaunchKernelGGL(k_table_grad_gather, dim3(nb(E * E * E, 32)), dim3(256), 0, st, part, m3, noff, sp,
                     offs, q, C, scale, g);
  return hipGetLastError();
}
}  // namespace

size_t table_grad_partial_doubles(int n, int m, int q, int noff) {
  const size_t S = 2 * q - 1;
  return (size_t)m * m * m * noff * grad_splits(n, m, noff) * S * S * S;
}

hipError_t table_grad(int n, int m, int q, int noff, const int* offs, const void* lam,
                      const void* M, int fp64, int C, double* part, double* g, hipStream_t st) {
  return grad<false>(n, m, q, noff, offs, lam, M, fp64, C, 1.0, part, g, st);
}

hipError_t mesh_table_grad(int n, int m, int q, int noff, const int* offs, const float* lam, const float* M,
                           int C, double scale, double* part, double* g, hipStream_t st) {
  return grad<true>(n, m, q, noff, offs, lam, M, 0, C, scale, part, g, st);
}

hipError_t orbit_gather(const double* g, const double* g0, const int* ptr, const int* pos, int nu,
                        float* ddelta, hipStream_t st) {
  hipLaunchKernelGGL(k_orbit_gather, dim3(nb(nu, 4)), dim3(256), 0, st, g, g0, ptr, pos, nu,
                     ddelta);
  return hipGetLastError();
}

size_t mlp_backward_partial_floats(int n) { return (size_t)nb(n, kBwdEntries) * kMlpParams; }

hipError_t mlp_backward(const float* theta, const float* feats, const float* ddelta, int n,
                        float* part, float* grad, hipStream_t st) {
  const int nblk = (int)nb(n, kBwdEntries);
  hipLaunchKernelGGL(k_mlp_backward, dim3(nblk), dim3(256), 0, st, theta, feats, ddelta, n, part);
  hipLaunchKernelGGL(k_sum_partials, dim3(nb(kMlpParams, 64)), dim3(64), 0, st, part, nblk, grad);
  return hipGetLastError();
}

hipError_t adam_step(float* theta, float* m1, float* m2, float* grad, int n, float count,
                     float lr, int step, hipStream_t st) {
  hipLaunchKernelGGL(k_adam, dim3(nb(n, 256)), dim3(256), 0, st, theta, m1, m2, grad, n, count,
                     lr, 0.9f, 0.999f, 1e-8f, step);
  return hipGetLastError();
}

hipError_t add_into(float* dst, const float* src, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_add_into, dim3(nb(n, 256)), dim3(256), 0, st, dst, src, n);
  return hipGetLastError();
}

}  // namespace pfmm
