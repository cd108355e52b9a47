// Conversion between the canonical array-of-structures lexicographic layouts, complex
// (Lt, Lz, Ly, Lx, 4, 3, 3) for links and (Lt, Lz, Ly, Lx, 4, 3) for spinors, and the even-odd
// structure-of-arrays layouts of lattice.hpp. Both are copies, bound by HBM: each side
// is moved in 16-byte accesses to consecutive addresses, through a transposition in LDS.
// A workgroup holds a run of consecutive sites (64, or 128 in FP32: the sites of 32 or 64
// checkerboard indices at both parities, so that a run of an element plane is 512 bytes).
// One thread per link without LDS reads the canonical side at a stride of a link and, in
// FP32, writes the planes in pieces of 64 bytes: at 32^3 x 64 pack and unpack took 266 and
// 393 us in FP32 (4.5 and 3.1 TB/s), 539 and 571 us in FP64; now 233 and 230 us, 460 and
// 449 us, 5.2 to 5.4 TB/s (a large copy: 5.1). Spinors: FP32 78 and 101 -> 76 and 77 us, FP64 183
// and 179 -> 154 and 148 us.
#include "kernels.hpp"

namespace sym {
namespace {

// NC complex components per site, in groups of G that share a (group, parity) block:
// component e = group * G + c of site (p, cb) is at ((group * 2 + p) * G + c) * Vh + cb.
template <typename T, int NC, int G, bool PACK>
__global__ __launch_bounds__(kBlock) void layout_kernel(Geom g, const T* __restrict__ src, T* __restrict__ dst) {
  constexpr int kCx = 16 / (int)sizeof(cx<T>);          // complex numbers per access
  constexpr int kSites = sizeof(T) == 4 ? 128 : 64;     // sites per workgroup
  constexpr int kRow = NC + 1;                          // LDS row of a site (+1: spreads the banks)
  constexpr int kQuads = kSites / 2 / kCx;              // accesses per run of a plane
  struct alignas(16) Unit {
    cx<T> v[kCx];
  };
  static_assert(NC % kCx == 0, "a site is whole accesses");
  __shared__ cx<T> buf[kSites * kRow];
  const int s0 = (int)blockIdx.x * kSites;
  const int ns = min(kSites, 2 * g.Vh - s0);  // a multiple of 16 (extents are even)
  const T* const aos_r = src + (size_t)s0 * NC * 2;
  T* const aos_w = dst + (size_t)s0 * NC * 2;

  if constexpr (PACK) {
    for (int i = threadIdx.x; i < ns * NC / kCx; i += kBlock) {
      const Unit u = reinterpret_cast<const Unit*>(aos_r)[i];
#pragma unroll
      for (int k = 0; k < kCx; ++k) {
        const int f = i * kCx + k;
        buf[f / NC * kRow + f % NC] = u.v[k];
      }
    }
    __syncthreads();
  }
  // plane runs: access q of plane (e, p) holds the checkerboard indices cb0 + kCx q ...
  const int cb0 = s0 >> 1, nq = ns / 2 / kCx;
  for (int i = threadIdx.x; i < 2 * NC * kQuads; i += kBlock) {
    const int q = i % kQuads, plane = i / kQuads, p = plane & 1, e = plane >> 1;
    if (q >= nq) continue;
    const size_t at = (size_t)((e / G * 2 + p) * G + e % G) * (size_t)g.Vh + (size_t)(cb0 + kCx * q);
    Unit u;
    if constexpr (!PACK) u = *reinterpret_cast<const Unit*>(reinterpret_cast<const cx<T>*>(src) + at);
#pragma unroll
    for (int k = 0; k < kCx; ++k) {
      // of the sites 2 cb and 2 cb + 1 the one of parity p
      const int cb = cb0 + kCx * q + k;
      int r = cb / g.Lxh;
      const int y = r % g.L[1];
      r /= g.L[1];
      const int x1 = (p + y + r % g.L[2] + r / g.L[2]) & 1;
      cx<T>& l = buf[(2 * (kCx * q + k) + x1) * kRow + e];
      if constexpr (PACK)
        u.v[k] = l;
      else
        l = u.v[k];
    }
    if constexpr (PACK) *reinterpret_cast<Unit*>(reinterpret_cast<cx<T>*>(dst) + at) = u;
  }
  if constexpr (!PACK) {
    __syncthreads();
    for (int i = threadIdx.x; i < ns * NC / kCx; i += kBlock) {
      Unit u;
#pragma unroll
      for (int k = 0; k < kCx; ++k) {
        const int f = i * kCx + k;
        u.v[k] = buf[f / NC * kRow + f % NC];
      }
      reinterpret_cast<Unit*>(aos_w)[i] = u;
    }
  }
}

template <typename T, int NC, int G>
hipError_t launch_layout(const Geom& g, const T* src, T* dst, bool pack, hipStream_t s) {
  constexpr int kSites = sizeof(T) == 4 ? 128 : 64;
  const unsigned blocks = (unsigned)((2 * g.Vh + kSites - 1) / kSites);
  if (pack)
    layout_kernel<T, NC, G, true><<<blocks, kBlock, 0, s>>>(g, src, dst);
  else
    layout_kernel<T, NC, G, false><<<blocks, kBlock, 0, s>>>(g, src, dst);
  return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_pack(const Geom& g, const T* aos, T* soa, hipStream_t s) {
  return launch_layout<T, 36, 9>(g, aos, soa, true, s);
}

template <typename T>
hipError_t launch_unpack(const Geom& g, const T* soa, T* aos, hipStream_t s) {
  return launch_layout<T, 36, 9>(g, soa, aos, false, s);
}

template <typename T>
hipError_t launch_spinor_layout(const Geom& g, const T* src, T* dst, bool pack, hipStream_t s) {
  return launch_layout<T, 12, 12>(g, src, dst, pack, s);
}

template hipError_t launch_pack<float>(const Geom&, const float*, float*, hipStream_t);
template hipError_t launch_pack<double>(const Geom&, const double*, double*, hipStream_t);
template hipError_t launch_unpack<float>(const Geom&, const float*, float*, hipStream_t);
template hipError_t launch_unpack<double>(const Geom&, const double*, double*, hipStream_t);
template hipError_t launch_spinor_layout<float>(const Geom&, const float*, float*, bool, hipStream_t);
template hipError_t launch_spinor_layout<double>(const Geom&, const double*, double*, bool, hipStream_t);

}  // namespace sym
