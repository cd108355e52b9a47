// Factored gauge force, single lattice: pass 1 (plaquette staples) and pass 2 (force)
// kernels over one lattice; the per-link device code is in factored.hpp.
#include "factored.hpp"

namespace sym {
namespace {

using factored::factored_link;
using factored::staples_site;

template <typename T>
__global__ __launch_bounds__(kBlock) void staples_kernel(Geom g, const T* __restrict__ U, T* __restrict__ S8,
                                                         int ntiles) {
  const SiteTile st = site_tile(g, blockIdx.x, ntiles);
  const int cb = st.chunk * kBlock + threadIdx.x;
  if (cb < g.Vh) staples_site(g, U, S8, st.p, cb);
}

// The workgroup's partials: the three deficit sums and, with KickOld and KickNew, the kinetic
// energy (both are written by those; either pointer may be null otherwise).
template <ForceOut MODE>
__device__ __forceinline__ void store_partials(double (&a)[4], double* __restrict__ partials,
                                               double* __restrict__ kin) {
  if constexpr (with_kinetic(MODE)) {
    block_sum<4>(a);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int k = 0; k < 3; ++k) partials[3 * (size_t)blockIdx.x + k] = a[k];
      kin[blockIdx.x] = a[3];
    }
  } else if (partials != nullptr) {
    double b[3] = {a[0], a[1], a[2]};
    block_sum_store<3>(b, partials + 3 * (size_t)blockIdx.x);
  }
}

template <typename T, ForceOut MODE>
__global__ __launch_bounds__(factored_links<T>()) void force_factored_kernel(Geom g, const T* __restrict__ U,
                                                                             const T* __restrict__ S8,
                                                                             T* __restrict__ out, double kick,
                                                                             double* __restrict__ partials,
                                                                             double* __restrict__ kin, Coeffs cf,
                                                                             int ntiles) {
  constexpr int N = factored_links<T>();
  const LinkSite lt = force_site<N>(g, blockIdx.x, ntiles, threadIdx.x);
  const int cb = lt.cb;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  if (cb < g.Vh) factored_link<T, MODE>(g, U, S8, out, kick, cf, lt.mu, lt.p, cb, a);
  store_partials<MODE>(a, partials, kin);
}

// Small lattices: a wave per site chunk and step of the staples, and eight waves per 64
// links (see the small-lattice part of factored.hpp).
template <typename T>
__global__ __launch_bounds__(64) void staples_small_kernel(Geom g, const T* __restrict__ U, T* __restrict__ S8) {
  const int role = blockIdx.x % kStapleRoles, tile = blockIdx.x / kStapleRoles;
  const int cb = (tile >> 1) * 64 + threadIdx.x;
  if (cb < g.Vh) factored::staple_one<0>(factored::site_ctx(g, U, S8, tile & 1, cb), role);
}

template <typename T, ForceOut MODE>
__global__ __launch_bounds__(64 * factored::kSmallWaves) void force_small_kernel(Geom g, const T* __restrict__ U,
                                                                                 const T* __restrict__ S8,
                                                                                 T* __restrict__ out, double kick,
                                                                                 double* __restrict__ partials,
                                                                                 double* __restrict__ kin,
                                                                                 Coeffs cf) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const LdsMats<T> m{reinterpret_cast<T*>(lds), (int)(threadIdx.x & 63)};
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int cb = (tile >> 3) * 64 + m.lane;
  const bool active = cb < g.Vh;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  factored::factored_link_small<T, MODE>(g, U, S8, out, kick, cf, tile & 3, (tile >> 2) & 1, active ? cb : 0, active,
                                         wave, m, a);
  store_partials<MODE>(a, partials, kin);
}

template <typename T, ForceOut MODE>
hipError_t launch_mode(const Geom& g, const T* U, const T* S8, T* out, double kick, double* partials, double* kin,
                       const Coeffs& c, hipStream_t s) {
  const int nt = factored_tiles<T>(g);
  if (force_is_small(g))
    force_small_kernel<T, MODE><<<nt, 64 * factored::kSmallWaves, factored::small_lds_bytes<T>(), s>>>(
        g, U, S8, out, kick, partials, kin, c);
  else
    // one or two waves per SIMD by registers (FP64, FP32); no LDS reservation: with
    // workgroups of one or two waves it would only take waves away
    force_factored_kernel<T, MODE><<<nt, factored_links<T>(), 0, s>>>(g, U, S8, out, kick, partials, kin, c, nt);
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_staples(const Geom& g, const T* U, T* S8, hipStream_t s) {
  if (staples_are_small<T>(g)) {
    const int chunks = (g.Vh + 63) / 64;
    staples_small_kernel<T><<<2 * chunks * kStapleRoles, 64, 0, s>>>(g, U, S8);
    return hipGetLastError();
  }
  const int nt = site_tiles(g);
  staples_kernel<T><<<nt, kBlock, 0, s>>>(g, U, S8, nt);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_force_factored(const Geom& g, const T* U, const T* S8, T* out, double kick, double* partials,
                                 double* kin, const Coeffs& c, ForceOut mode, hipStream_t s) {
  switch (mode) {
    case ForceOut::Store:
      return launch_mode<T, ForceOut::Store>(g, U, S8, out, kick, partials, kin, c, s);
    case ForceOut::Kick:
      return launch_mode<T, ForceOut::Kick>(g, U, S8, out, kick, partials, kin, c, s);
    case ForceOut::Grad:
      return launch_mode<T, ForceOut::Grad>(g, U, S8, out, kick, partials, kin, c, s);
    case ForceOut::KickOld:
      return launch_mode<T, ForceOut::KickOld>(g, U, S8, out, kick, partials, kin, c, s);
    default:
      return launch_mode<T, ForceOut::KickNew>(g, U, S8, out, kick, partials, kin, c, s);
  }
}

#ifndef SYM_ONLY_F64
template hipError_t launch_staples<float>(const Geom&, const float*, float*, hipStream_t);
#endif
#ifndef SYM_ONLY_F32
template hipError_t launch_staples<double>(const Geom&, const double*, double*, hipStream_t);
#endif
#ifndef SYM_ONLY_F64
template hipError_t launch_force_factored<float>(const Geom&, const float*, const float*, float*, double, double*,
                                                 double*, const Coeffs&, ForceOut, hipStream_t);
#endif
#ifndef SYM_ONLY_F32
template hipError_t launch_force_factored<double>(const Geom&, const double*, const double*, double*, double, double*,
                                                  double*, const Coeffs&, ForceOut, hipStream_t);
#endif

}  // namespace sym
