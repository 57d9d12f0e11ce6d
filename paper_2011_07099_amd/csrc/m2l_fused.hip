// The spectral zones' node transforms fused with the tree's transfers: the
// masses of a node are transformed by the workgroup that forms them (M2M or
// P2M), and a node's zone sums go from its inverse transform straight to its
// children (L2L) or its cells (L2P).  The arithmetic and its order are those of
// the separate kernels.
//
// These steps move little (a node's p^3 values and 16 (2p)^2 (p + 1) bytes of
// spectrum) and are bound by launches and latency in boxes of up to some 10^3
// nodes: four launches and round trips less out of ten in a tree of three
// levels.  A solve before / after: 64^3, p = 7 121 / 107 us, 64^3 in FP64 130 / 115,
// 128^3, p = 6 142 / 137, 32 mixed fields 2213 / 2111; boxes bound elsewhere (256^3,
// 512^3) neither gain nor lose.
#include "columns.h"
#include "spectral.h"

namespace pfmm {
namespace {

constexpr int kThreads = kColThreads;

constexpr int cmax(int a, int b) { return a > b ? a : b; }
// doubles of the two node transform buffers
template <int P>
constexpr int node_words() { return 4 * P * P * (P + 1); }

template <class TI, int P>
__global__ __launch_bounds__(kThreads) void k_m2m_fwd(const TI* __restrict__ Mc, double* __restrict__ Mp,
                                                       Weights Tw, int np, double2* __restrict__ spec) {
  constexpr int P3 = P * P * P;
  __shared__ double2 lds[cmax(pair_words<P>(), node_words<P>()) / 2];
  __shared__ double mass[P3];
  const int64_t nn = (int64_t)np * np * np, node = xcd_node(blockIdx.x, nn);
  m2m_block<TI, double, P>(Mc, Tw.d, np, (int)node, reinterpret_cast<double*>(lds), [&](int i, double v) {
    mass[i] = v;
    Mp[node * P3 + i] = v;
  });
  __syncthreads();
  node_fwd_block<P, kThreads>([&](int i) { return mass[i]; }, node, nn, spec, lds, lds + P * P * (P + 1));
}

template <class TR, int S, int P>
__global__ __launch_bounds__(kThreads) void k_p2m_fwd(const TR* __restrict__ rho, double* __restrict__ M,
                                                       Weights Aw, int N, double h3, int vec,
                                                       double2* __restrict__ spec) {
  constexpr int P3 = P * P * P;
  __shared__ double2 lds[(cmax(p2m_col_words<S, P>(), node_words<P>()) + 1) / 2];
  __shared__ double mass[P3];
  const int nL = N / S;
  const int64_t nn = (int64_t)nL * nL * nL, node = xcd_node(blockIdx.x, nn);
  p2m_block<TR, double, S, P>(rho, Aw.d, N, (int)node, h3, vec, reinterpret_cast<double*>(lds),
                              [&](int i, double v) {
    mass[i] = v;
    M[node * P3 + i] = v;
  });
  __syncthreads();
  node_fwd_block<P, kThreads>([&](int i) { return mass[i]; }, node, nn, spec, lds, lds + P * P * (P + 1));
}

template <class TO, int P>
__global__ __launch_bounds__(kThreads) void k_inv_l2l(const double2* __restrict__ out, double* __restrict__ Pl,
                                                       int accumulate, TO* __restrict__ Pc, Weights Tw, int np) {
  constexpr int P3 = P * P * P;
  __shared__ double2 lds[cmax(pair_words<P>(), node_words<P>()) / 2];
  __shared__ double loc[P3];
  const int64_t nn = (int64_t)np * np * np, node = xcd_node(blockIdx.x, nn);
  double* dst = Pl + node * P3;
  node_inv_block<P, kThreads>(out, node, nn, lds, lds + P * P * (P + 1), [&](int i, double v) {
    if (accumulate) v = dst[i] + v;
    dst[i] = loc[i] = v;
  });
  __syncthreads();
  l2l_block<TO, double, P>([&](int i) { return loc[i]; }, Pc, Tw.d, np, (int)node, 0,
                           reinterpret_cast<double*>(lds));
}

template <class TP, int S, int P>
__global__ __launch_bounds__(kThreads) void k_inv_l2p(const double2* __restrict__ out, double* __restrict__ Pl,
                                                       int accumulate, TP* __restrict__ phi, Weights Aw, int N) {
  constexpr int P3 = P * P * P;
  __shared__ double2 lds[(cmax(l2p_col_words<S, P>(), node_words<P>()) + 1) / 2];
  __shared__ double loc[P3];
  const int nL = N / S;
  const int64_t nn = (int64_t)nL * nL * nL, node = xcd_node(blockIdx.x, nn);
  double* dst = Pl + node * P3;
  node_inv_block<P, kThreads>(out, node, nn, lds, lds + P * P * (P + 1), [&](int i, double v) {
    if (accumulate) v = dst[i] + v;
    dst[i] = loc[i] = v;
  });
  __syncthreads();
  l2p_block<TP, double, S, P>([&](int i) { return loc[i]; }, phi, Aw.d, Aw.d, Aw.d, 1.0, N, (int)node, 1,
                              reinterpret_cast<double*>(lds));
}

template <int P, class TR>
hipError_t p2m_fwd(const TR* rho, double* M, Weights A, int N, int s, double h3, double2* spec, hipStream_t st) {
  const unsigned g = (unsigned)(N / s) * (N / s) * (N / s);
  const int vec = ((uintptr_t)rho & 15) == 0;
  if (s == 16)
    k_p2m_fwd<TR, 16, P><<<g, kThreads, 0, st>>>(rho, M, A, N, h3, vec, spec);
  else if (s == 8)
    k_p2m_fwd<TR, 8, P><<<g, kThreads, 0, st>>>(rho, M, A, N, h3, vec, spec);
  else if (s == 4)
    k_p2m_fwd<TR, 4, P><<<g, kThreads, 0, st>>>(rho, M, A, N, h3, vec, spec);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int P, class TP>
hipError_t inv_l2p(const double2* out, double* Pl, int accumulate, TP* phi, Weights A, int N, int s,
                   hipStream_t st) {
  const unsigned g = (unsigned)(N / s) * (N / s) * (N / s);
  if (s == 16)
    k_inv_l2p<TP, 16, P><<<g, kThreads, 0, st>>>(out, Pl, accumulate, phi, A, N);
  else if (s == 8)
    k_inv_l2p<TP, 8, P><<<g, kThreads, 0, st>>>(out, Pl, accumulate, phi, A, N);
  else if (s == 4)
    k_inv_l2p<TP, 4, P><<<g, kThreads, 0, st>>>(out, Pl, accumulate, phi, A, N);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

bool fused_zones(const M2LSpectral* f, int p) { return f && p >= 3 && p <= 8; }

hipError_t fused_m2m(const M2LSpectral* f, int l, const void* Mc, int c64, double* Mp, Weights T,
                     hipStream_t st) {
  const int np = 1 << l;
  return with_p<3, 8>(f->p, [&](auto Pc) {
    constexpr int P = decltype(Pc)::value;
    const unsigned g = (unsigned)np * np * np;
    if (c64)
      k_m2m_fwd<double, P><<<g, kThreads, 0, st>>>((const double*)Mc, Mp, T, np, f->spec[l]);
    else
      k_m2m_fwd<float, P><<<g, kThreads, 0, st>>>((const float*)Mc, Mp, T, np, f->spec[l]);
    return hipGetLastError();
  });
}

hipError_t fused_p2m(const M2LSpectral* f, int l, const void* rho, int rho64, double* M, Weights A, int N, int s,
                     double h3, hipStream_t st) {
  return with_p<3, 8>(f->p, [&](auto Pc) {
    constexpr int P = decltype(Pc)::value;
    return rho64 ? p2m_fwd<P>((const double*)rho, M, A, N, s, h3, f->spec[l], st)
                 : p2m_fwd<P>((const float*)rho, M, A, N, s, h3, f->spec[l], st);
  });
}

hipError_t fused_l2l(const M2LSpectral* f, int l, double* Pl, int accumulate, void* Pc, int c64, Weights T,
                     hipStream_t st) {
  const int np = 1 << l;
  return with_p<3, 8>(f->p, [&](auto Pn) {
    constexpr int P = decltype(Pn)::value;
    const unsigned g = (unsigned)np * np * np;
    if (c64)
      k_inv_l2l<double, P><<<g, kThreads, 0, st>>>(f->out, Pl, accumulate, (double*)Pc, T, np);
    else
      k_inv_l2l<float, P><<<g, kThreads, 0, st>>>(f->out, Pl, accumulate, (float*)Pc, T, np);
    return hipGetLastError();
  });
}

hipError_t fused_l2p(const M2LSpectral* f, int l, double* Pl, int accumulate, void* phi, int phi64, Weights A,
                     int N, int s, hipStream_t st) {
  (void)l;
  return with_p<3, 8>(f->p, [&](auto Pc) {
    constexpr int P = decltype(Pc)::value;
    return phi64 ? inv_l2p<P>(f->out, Pl, accumulate, (double*)phi, A, N, s, st)
                 : inv_l2p<P>(f->out, Pl, accumulate, (float*)phi, A, N, s, st);
  });
}

}  // namespace pfmm
