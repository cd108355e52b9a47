// Fat-link smearing (asqtad / HISQ) and its path force: kernels and launchers.
// The per-link device code and the derivation are in fat.hpp.
#include "fat.hpp"

namespace sym {

using fat::Ctx;
using fat::FatCoeffs;
using fat::Fields;

namespace {

// Tiles of the passes that read intermediate fields at neighbouring links: the walk of the
// force pass (force_tile) with the parity fastest, so that the two parities of a chunk, which
// read each other's fields, run side by side. On large lattices these passes are bound by field
// data from beyond the L2.
__device__ __forceinline__ LinkTile fat_tile(const Geom& g, int linear, int ntiles) {
  LinkTile lt = force_tile(g, linear, ntiles, kBlock);
  const int q = lt.p * 4 + lt.mu;
  lt.p = q & 1;
  lt.mu = q >> 1;
  return lt;
}

// ... of FK2, FK3 and (BK2) the reverse pass, above 2^17 sites. Against direction fastest in
// t-fastest slabs (link_tile), us: FP32 32^4 FK2 1293 -> 1213, BK2 1423 -> 1378; 20^3 x 40, where the
// walk does not apply and only the parity moves, FK3 231 -> 226, FK2 394 -> 386; FP64 32^4 FK3
// 1327 -> 1260, FK2 2214 -> 2182, 24^3 x 48 847 -> 822 and 1471 -> 1432. Below, much of the fields is
// in the Infinity Cache and link_tile is as fast or faster: 32 x 16^3 FP32 FK3 91 and 93, BK2
// 160 and 163, FP64 FK2 248 and 253, FK3 162 and 166, BK2 291 and 300. BK2 in FP64 gains by the
// walk (16 x 32 x 16 x 64 1276 -> 1220, 32^4 2606 -> 2578) but not by the parity alone (16^2 x 32^2
// 567 and 582, 20^3 x 40 801 and 805). FK1, which reads links only, was slower in this order
// throughout (1.06 and 1.12 ms in FP32 at 32^3 x 64), BK3 no faster.
constexpr int kFatTileVh = 1 << 16;

template <typename T, bool BK2>
__device__ __forceinline__ LinkTile field_tile(const Geom& g, int linear, int ntiles) {
  const bool walk_only = BK2 && sizeof(T) == 8;
  if (g.Vh <= kFatTileVh || (walk_only && !planes_are_chunks(g, kBlock))) return link_tile(g, linear, ntiles);
  return fat_tile(g, linear, ntiles);
}

// The link of a thread of the gradient gather GK, which reads the most fields: a workgroup of
// four waves takes 64 links in each of four z-neighbouring planes (or 128 in each of two),
// whose transports along z then meet in one CU's L1 and at the same time in the L2; parity
// fastest, then direction, t through the XCD's slab, y, z. Against fat_tile, FP32: 32^3 x 64
// 6.67 -> 6.43, 32 x 24^2 x 32 1.80 -> 1.73 ms; against link_tile, FP64: 32^4 6.27 -> 5.55,
// 32 x 24^2 x 32 3.49 -> 3.15, 32 x 16 x 32 x 16 1.50 -> 1.40, 32 x 16^2 x 48 2.37 -> 2.34 ms. FP64
// planes below a workgroup (16^3 x 32) take 0.685 ms in fours, 0.665 in twos, which is where
// they were. Planes that are not whole runs of 64 gain nothing from eight planes of 32 links
// (FP64 24^4 1.94 ms either way) and keep fat_tile (FP32: 24^3 x 48 2.13 -> 2.11 ms) and link_tile
// (FP64). The other passes lose by the blocks
// on some lattices what they gain on others (FP64 FK2 and BK2 at 32^4 2.18 -> 2.06 and 2.59 ->
// 2.48, at 32 x 16^2 x 48 0.79 -> 0.83 and 0.93 -> 1.03 ms).
template <typename T>
__device__ __forceinline__ int gk_planes(const Geom& g) {
  const int plane = g.Lxh * g.L[1];
  if (plane % 64 == 0 && g.L[2] % 4 == 0 && (sizeof(T) == 4 || plane >= kBlock)) return 4;
  return plane % 128 == 0 ? 2 : 0;  // Lz is even
}

template <typename T>
__device__ __forceinline__ LinkSite gk_site(const Geom& g, int linear, int ntiles) {
  const int lane = threadIdx.x;
  const int m = gk_planes<T>(g);
  if (m == 0) {
    const LinkTile lt = sizeof(T) == 4 ? fat_tile(g, linear, ntiles) : link_tile(g, linear, ntiles);
    return LinkSite{lt.mu, lt.p, lt.chunk * kBlock + lane};
  }
  const int tile = xcd_tile(linear, ntiles);
  const int run = kBlock / m, plane = g.Lxh * g.L[1];
  const int slab = (g.L[3] + 7) >> 3, Ly = plane / run, Lz = g.L[2] / m, Lt = g.L[3];
  int k = tile >> 3;
  const int t0 = k / (slab * Lz * Ly) * slab;
  const int tn = min(slab, Lt - t0);
  k -= t0 * Lz * Ly;
  const int z = k / (Ly * tn);
  k -= z * Ly * tn;
  const int y = k / tn, t = t0 + k - y * tn;
  const int cb = plane * (m * z + lane / run + g.L[2] * t) + run * y + lane % run;
  return LinkSite{(tile >> 1) & 3, tile & 1, cb};
}

template <typename T>
__global__ __launch_bounds__(kBlock) void fat_fk1_kernel(Geom g, const T* __restrict__ U, Fields<T> w, FatCoeffs cf,
                                                          int ntiles) {
  const LinkTile lt = link_tile(g, blockIdx.x, ntiles);
  const int cb = lt.chunk * kBlock + threadIdx.x;
  if (cb >= g.Vh) return;
  Ctx<T> c;
  fat::make_ctx(g, U, lt.mu, lt.p, cb, c);
  fat::fk1_step<1>(c, w, T(cf.c[2]), T(cf.c[3]), cb);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void fat_fk2_kernel(Geom g, const T* __restrict__ U, Fields<T> w, FatCoeffs cf,
                                                          int ntiles) {
  const LinkTile lt = field_tile<T, false>(g, blockIdx.x, ntiles);
  const int cb = lt.chunk * kBlock + threadIdx.x;
  if (cb >= g.Vh) return;
  Ctx<T> c;
  fat::make_ctx(g, U, lt.mu, lt.p, cb, c);
  // transport direction outermost (two_out), both precisions; FP64 holds the three
  // accumulators in VGPRs and AGPRs at one wave per SIMD (6.05 -> 4.71 ms at 32^3 x 64
  // against one M at a time)
  su3<T> acc[3];
  const su3<T> u = c.template u<0, 0, 0, 0, 0>();
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    acc[k] = u;
    fat::scale(acc[k], T(cf.c[1]));
  }
  SYM_FAT_FENCE();
  fat::two_out<1, false>(acc, c, static_cast<const T*>(w.inner));
  fat::launder(c);
  SYM_FAT_FENCE();
  fat::store_m<1>(acc[0], c, w, T(cf.c[4]), cb);
  SYM_FAT_FENCE();
  fat::store_m<2>(acc[1], c, w, T(cf.c[4]), cb);
  SYM_FAT_FENCE();
  fat::store_m<3>(acc[2], c, w, T(cf.c[4]), cb);
}

// W = cN U_{x,mu} U_{x+mu,mu} U_{x+2mu,mu}
template <typename T>
__device__ __forceinline__ su3<T> naik_link(const Ctx<T>& c, const FatCoeffs& cf) {
  su3<T> nk = mul<false, false>(c.template u<0, 0, 0, 0, 0>(), c.template u<1, 0, 0, 0, 0>());
  nk = mul<false, false>(nk, c.template u<2, 0, 0, 0, 0>());
  fat::scale(nk, T(cf.c[5]));
  return nk;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void fat_fk3_kernel(Geom g, const T* __restrict__ U, Fields<T> w,
                                                          T* __restrict__ V, T* __restrict__ W, FatCoeffs cf,
                                                          int ntiles) {
  const LinkTile lt = field_tile<T, false>(g, blockIdx.x, ntiles);
  const int cb = lt.chunk * kBlock + threadIdx.x;
  if (cb >= g.Vh) return;
  Ctx<T> c;
  fat::make_ctx(g, U, lt.mu, lt.p, cb, c);
  su3<T> acc = c.template u<0, 0, 0, 0, 0>();
  fat::scale(acc, T(cf.c[0]));
  fat::fk3_step<1>(acc, c, w);
  store_link(block_ptr(V, lt.mu, lt.p, g.Vh), g.Vh, cb, acc);
  if (W != nullptr) {
    fat::launder(c);
    store_link(block_ptr(W, lt.mu, lt.p, g.Vh), g.Vh, cb, naik_link(c, cf));
  }
}

// FP32: six waves per SIMD (80 VGPRs, no spills): 1.26 -> 1.16 ms at 32^3 x 64
template <typename T>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 6 : 1))) void fat_bk3_kernel(Geom g, const T* __restrict__ U, const T* __restrict__ GV,
                                                          Fields<T> w, int ntiles) {
  const LinkTile lt = link_tile(g, blockIdx.x, ntiles);
  const int cb = lt.chunk * kBlock + threadIdx.x;
  if (cb >= g.Vh) return;
  Ctx<T> c;
  fat::make_ctx(g, U, lt.mu, lt.p, cb, c);
  fat::bk3_step<1>(c, GV, w, cb);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void fat_bk2_kernel(Geom g, const T* __restrict__ U, const T* __restrict__ GV,
                                                          Fields<T> w, FatCoeffs cf, int ntiles) {
  const LinkTile lt = field_tile<T, true>(g, blockIdx.x, ntiles);
  const int cb = lt.chunk * kBlock + threadIdx.x;
  if (cb >= g.Vh) return;
  Ctx<T> c;
  fat::make_ctx(g, U, lt.mu, lt.p, cb, c);
  // D = c1 GV + c3 sum_k gmid_k + c5 sum_m g_inner_m
  su3<T> dsum = c.template f<0, 0, 0, 0, 0>(GV, 1, 0);
  fat::scale(dsum, T(cf.c[0]));
  for (int k = 0; k < 3; ++k) axpy(dsum, T(cf.c[1]), c.template f<0, 0, 0, 0, 0>(w.gmid, 3, k));
  SYM_FAT_FENCE();
  // transport direction outermost, both precisions (FP64: 6.78 -> 5.50 ms at 32^3 x 64)
  su3<T> gi[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) set_zero(gi[k]);
  fat::two_out<1, true>(gi, c, static_cast<const T*>(w.gmid));
  fat::launder(c);
  const T c5 = T(cf.c[2]), c7 = T(cf.c[3]), cL = T(cf.c[4]);
  SYM_FAT_FENCE();
  fat::store_gt<1>(gi[0], c, GV, w, c7, cL, cb);
  SYM_FAT_FENCE();
  fat::store_gt<2>(gi[1], c, GV, w, c7, cL, cb);
  SYM_FAT_FENCE();
  fat::store_gt<3>(gi[2], c, GV, w, c7, cL, cb);
#pragma unroll
  for (int m = 0; m < 3; ++m) axpy(dsum, c5, gi[m]);
  fat::store_slot(w.D, 1, 0, lt.mu, lt.p, g.Vh, cb, dsum);
}

// The terms of a thin link's own chain: the direct terms D, the transports of U_nu itself,
// and the Naik terms.
template <typename T>
__device__ __forceinline__ su3<T> own_terms(const Ctx<T>& c, const T* GW, const Fields<T>& w, const FatCoeffs& cf) {
  su3<T> acc = c.template f<0, 0, 0, 0, 0>(w.D, 1, 0);
  SYM_FAT_FENCE();
  fat::gk_pull<1>(acc, c, w);

  if (GW != nullptr) {
    // W_{y-k nu} = cN U_{y-k nu,nu} U_{y-(k-1)nu,nu} U_{y-(k-2)nu,nu} for k = 0, 1, 2
    Ctx<T> cc = c;
    fat::launder(cc);
    const su3<T> u1 = cc.template u<1, 0, 0, 0, 0>(), u2 = cc.template u<2, 0, 0, 0, 0>();
    su3<T> t = mul<false, true>(cc.template f<0, 0, 0, 0, 0>(GW, 1, 0), u2);
    su3<T> nk = mul<false, true>(t, u1);
    const su3<T> um1 = cc.template u<-1, 0, 0, 0, 0>();
    t = mul<true, false>(um1, cc.template f<-1, 0, 0, 0, 0>(GW, 1, 0));
    mac<false, true>(nk, t, u1);
    t = mul<true, true>(um1, cc.template u<-2, 0, 0, 0, 0>());
    mac<false, false>(nk, t, cc.template f<-2, 0, 0, 0, 0>(GW, 1, 0));
    axpy(acc, T(cf.c[5]), nk);
    SYM_FAT_FENCE();
  }
  return acc;
}

// The gradient acc of link (mu, p, cb) to `out`, or the force of it.
template <int MODE, typename T>
__device__ __forceinline__ void store_result(const su3<T>& acc, const Ctx<T>& c0, T* out, int cb) {
  Ctx<T> c = c0;
  fat::launder(c);
  cx<T>* dst = block_ptr(out, c.ax[0], c.p, c.Vh);
  if constexpr (MODE == 0) {
    store_link(dst, c.Vh, cb, acc);
  } else {
    // G = -(1/2)(U grad^dagger)_TA, the force in the convention of the gauge force
    const su3<T> b = mul<false, true>(c.template u<0, 0, 0, 0, 0>(), acc);
    store_link(dst, c.Vh, cb, ta_scaled(b, T(-0.5)));
  }
}

// Gradient (or force) of the thin link (y, nu): the terms of its own chain, and the deposits
// of the transports along nu of the other chains.
template <typename T, int MODE>
__global__ __launch_bounds__(kBlock) void fat_gk_kernel(Geom g, const T* __restrict__ U, const T* __restrict__ GV,
                                                         const T* __restrict__ GW, Fields<T> w, T* __restrict__ out,
                                                         FatCoeffs cf, int ntiles) {
  const LinkSite lt = gk_site<T>(g, blockIdx.x, ntiles);
  const int cb = lt.cb;
  if (cb >= g.Vh) return;
  Ctx<T> c;
  fat::make_ctx(g, U, lt.mu, lt.p, cb, c);
  su3<T> acc = own_terms(c, GW, w, cf);
  fat::gk_chains<1>(acc, c, GV, w);
  store_result<MODE>(acc, c, out, cb);
}

// ------------------------------------------------------------ small lattices
// With one wave per 64 links small lattices leave most SIMDs empty and wait for one wave's
// serial products. Here a workgroup of three or four waves shares 64 links (one per lane of
// every wave), with partial sums in LDS, so that the results are those of the whole-link form
// to rounding: each wave's sum starts from zero and the sums are added. That pays up to 512
// workgroups (kFatSmallTiles), which in FP64 run in two rounds: FK2, BK2 and GK take more than
// 256 registers and so one workgroup per CU.
// Path force, before -> now: FP32 4^4 81 -> 42 us, 8^4 104 -> 47, 8^3 x 16 (512 workgroups) 107 -> 65;
// FP64 4^4 90 -> 46 us, 8^4 124 -> 54, 8^3 x 16 136 -> 98. With 1024 workgroups (8^2 x 16^2) it would
// be 117 -> 117 us in FP32 and 172 -> 194 us in FP64.

// The link of a lane and its wave.
template <typename T>
struct SmallLink {
  Ctx<T> c;
  int cb, wave;
  bool active;  // false past the end of the lattice: such lanes only take part in barriers
};

template <typename T>
__device__ __forceinline__ SmallLink<T> small_link(const Geom& g, const T* U) {
  SmallLink<T> s;
  s.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  s.cb = (tile >> 3) * 64 + (threadIdx.x & 63);
  s.active = s.cb < g.Vh;
  s.cb = s.active ? s.cb : 0;
  fat::make_ctx(g, U, tile & 3, (tile >> 2) & 1, s.cb, s.c);
  return s;
}

// FK1 and BK3: wave K-1 writes slot K.
template <typename T>
__global__ __launch_bounds__(192) void fat_fk1_small_kernel(Geom g, const T* __restrict__ U, Fields<T> w, FatCoeffs cf) {
  const SmallLink<T> s = small_link(g, U);
  if (!s.active) return;
  const T c5 = T(cf.c[2]), c7 = T(cf.c[3]);
  if (s.wave == 0)
    fat::fk1_one<1>(s.c, w, c5, c7, s.cb);
  else if (s.wave == 1)
    fat::fk1_one<2>(s.c, w, c5, c7, s.cb);
  else
    fat::fk1_one<3>(s.c, w, c5, c7, s.cb);
}

template <typename T>
__global__ __launch_bounds__(192) void fat_bk3_small_kernel(Geom g, const T* __restrict__ U, const T* __restrict__ GV,
                                                            Fields<T> w) {
  const SmallLink<T> s = small_link(g, U);
  if (!s.active) return;
  if (s.wave == 0)
    fat::bk3_one<1>(s.c, GV, w, s.cb);
  else if (s.wave == 1)
    fat::bk3_one<2>(s.c, GV, w, s.cb);
  else
    fat::bk3_one<3>(s.c, GV, w, s.cb);
}

// FK2 and BK2, first half: wave J-1 forms the transports along ax[J], which serve the two
// outputs k other than J-1, into LDS.
constexpr int kTransports = 6;
constexpr int transport_slot(int J, int k) { return 2 * (J - 1) + (k > J - 1 ? k - 1 : k); }
template <int J, bool BACK, typename T>
__device__ __forceinline__ void small_two_out(const SmallLink<T>& s, const T* F, const LdsMats<T>& m) {
  su3<T> acc[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) set_zero(acc[k]);
  fat::two_out_one<J, BACK>(acc, s.c, F);
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (k != J - 1) m.put(transport_slot(J, k), acc[k]);
}
template <bool BACK, typename T>
__device__ __forceinline__ void small_transports(const SmallLink<T>& s, const T* F, const LdsMats<T>& m) {
  if (s.active) {
    if (s.wave == 0)
      small_two_out<1, BACK>(s, F, m);
    else if (s.wave == 1)
      small_two_out<2, BACK>(s, F, m);
    else if (s.wave == 2)
      small_two_out<3, BACK>(s, F, m);
  }
  __syncthreads();
}
// ... second half: the sum for output `k` in order of J.
template <typename T>
__device__ __forceinline__ void small_sum(su3<T>& acc, int k, const LdsMats<T>& m) {
#pragma unroll
  for (int J = 1; J <= 3; ++J)
    if (J - 1 != k) add(acc, m.get(transport_slot(J, k)));
}

template <int K, typename T>
__device__ __forceinline__ void small_m(const SmallLink<T>& s, const Fields<T>& w, const FatCoeffs& cf,
                                        const LdsMats<T>& m) {
  su3<T> acc = s.c.template u<0, 0, 0, 0, 0>();
  fat::scale(acc, T(cf.c[1]));
  small_sum(acc, K - 1, m);
  fat::store_m<K>(acc, s.c, w, T(cf.c[4]), s.cb);
}

template <typename T>
__global__ __launch_bounds__(192) void fat_fk2_small_kernel(Geom g, const T* __restrict__ U, Fields<T> w, FatCoeffs cf) {
  __shared__ T lds[kTransports * 18 * 64];
  const SmallLink<T> s = small_link(g, U);
  const LdsMats<T> m{lds, (int)(threadIdx.x & 63)};
  small_transports<false>(s, static_cast<const T*>(w.inner), m);
  if (!s.active) return;
  if (s.wave == 0)
    small_m<1>(s, w, cf, m);
  else if (s.wave == 1)
    small_m<2>(s, w, cf, m);
  else
    small_m<3>(s, w, cf, m);
}

template <int M, typename T>
__device__ __forceinline__ void small_gt(const SmallLink<T>& s, const T* GV, const Fields<T>& w, const FatCoeffs& cf,
                                         const LdsMats<T>& m) {
  su3<T> gi;
  set_zero(gi);
  small_sum(gi, M - 1, m);
  fat::store_gt<M>(gi, s.c, GV, w, T(cf.c[3]), T(cf.c[4]), s.cb);
}

template <typename T>
__global__ __launch_bounds__(256) void fat_bk2_small_kernel(Geom g, const T* __restrict__ U, const T* __restrict__ GV,
                                                            Fields<T> w, FatCoeffs cf) {
  __shared__ T lds[kTransports * 18 * 64];
  const SmallLink<T> s = small_link(g, U);
  const LdsMats<T> m{lds, (int)(threadIdx.x & 63)};
  small_transports<true>(s, static_cast<const T*>(w.gmid), m);
  if (!s.active) return;
  if (s.wave == 0) {
    small_gt<1>(s, GV, w, cf, m);
  } else if (s.wave == 1) {
    small_gt<2>(s, GV, w, cf, m);
  } else if (s.wave == 2) {
    small_gt<3>(s, GV, w, cf, m);
  } else {
    // D = c1 GV + c3 sum_k gmid_k + c5 sum_m g_inner_m
    su3<T> d = s.c.template f<0, 0, 0, 0, 0>(GV, 1, 0);
    fat::scale(d, T(cf.c[0]));
    for (int k = 0; k < 3; ++k) axpy(d, T(cf.c[1]), s.c.template f<0, 0, 0, 0, 0>(w.gmid, 3, k));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      su3<T> gi;
      set_zero(gi);
      small_sum(gi, k, m);
      axpy(d, T(cf.c[2]), gi);
    }
    fat::store_slot(w.D, 1, 0, s.c.ax[0], s.c.p, g.Vh, s.cb, d);
  }
}

// FK3: waves 0..2 the transports along ax[1..3], wave 3 the Naik link.
template <typename T>
__global__ __launch_bounds__(256) void fat_fk3_small_kernel(Geom g, const T* __restrict__ U, Fields<T> w,
                                                            T* __restrict__ V, T* __restrict__ W, FatCoeffs cf) {
  __shared__ T lds[2 * 18 * 64];
  const SmallLink<T> s = small_link(g, U);
  const LdsMats<T> m{lds, (int)(threadIdx.x & 63)};
  su3<T> acc;
  set_zero(acc);
  if (s.active) {
    if (s.wave == 0) {
      acc = s.c.template u<0, 0, 0, 0, 0>();
      fat::scale(acc, T(cf.c[0]));
      fat::fk3_one<1>(acc, s.c, w);
    } else if (s.wave == 1) {
      fat::fk3_one<2>(acc, s.c, w);
      m.put(0, acc);
    } else if (s.wave == 2) {
      fat::fk3_one<3>(acc, s.c, w);
      m.put(1, acc);
    } else if (W != nullptr) {
      store_link(block_ptr(W, s.c.ax[0], s.c.p, g.Vh), g.Vh, s.cb, naik_link(s.c, cf));
    }
  }
  __syncthreads();
  if (!s.active || s.wave != 0) return;
  add(acc, m.get(0));
  add(acc, m.get(1));
  store_link(block_ptr(V, s.c.ax[0], s.c.p, g.Vh), g.Vh, s.cb, acc);
}

// GK: wave 0 the own terms, waves 1..3 the deposits from the chains of ax[1..3].
template <typename T, int MODE>
__global__ __launch_bounds__(256) void fat_gk_small_kernel(Geom g, const T* __restrict__ U, const T* __restrict__ GV,
                                                           const T* __restrict__ GW, Fields<T> w, T* __restrict__ out,
                                                           FatCoeffs cf) {
  __shared__ T lds[3 * 18 * 64];
  const SmallLink<T> s = small_link(g, U);
  const LdsMats<T> m{lds, (int)(threadIdx.x & 63)};
  su3<T> acc;
  set_zero(acc);
  if (s.active) {
    if (s.wave == 0)
      acc = own_terms(s.c, GW, w, cf);
    else if (s.wave == 1)
      fat::gk_chain<1>(acc, s.c, GV, w);
    else if (s.wave == 2)
      fat::gk_chain<2>(acc, s.c, GV, w);
    else
      fat::gk_chain<3>(acc, s.c, GV, w);
    if (s.wave > 0) m.put(s.wave - 1, acc);
  }
  __syncthreads();
  if (!s.active || s.wave != 0) return;
#pragma unroll
  for (int k = 0; k < 3; ++k) add(acc, m.get(k));
  store_result<MODE>(acc, s.c, out, s.cb);
}

}  // namespace

template <typename T>
hipError_t launch_fat_fk3(const Geom& g, const T* U, T* V, T* W, const FatCoeffs& c, const Fields<T>& w,
                          hipStream_t s) {
  if (fat_is_small(g)) {
    fat_fk3_small_kernel<T><<<link_tiles(g, 64), 256, 0, s>>>(g, U, w, V, W, c);
    return hipGetLastError();
  }
  const int nt = link_tiles(g);
  fat_fk3_kernel<T><<<nt, kBlock, 0, s>>>(g, U, w, V, W, c, nt);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fat_stage(int stage, const Geom& g, const T* U, const T* GV, const T* GW, T* out, int mode,
                            const FatCoeffs& c, const Fields<T>& w, hipStream_t s) {
  if (fat_is_small(g)) {
    const int n = link_tiles(g, 64);
    switch (stage) {
      case 0:
        fat_fk1_small_kernel<T><<<n, 192, 0, s>>>(g, U, w, c);
        break;
      case 1:
        fat_fk2_small_kernel<T><<<n, 192, 0, s>>>(g, U, w, c);
        break;
      case 2:
        fat_bk3_small_kernel<T><<<n, 192, 0, s>>>(g, U, GV, w);
        break;
      case 3:
        fat_bk2_small_kernel<T><<<n, 256, 0, s>>>(g, U, GV, w, c);
        break;
      default:
        if (mode == 0)
          fat_gk_small_kernel<T, 0><<<n, 256, 0, s>>>(g, U, GV, GW, w, out, c);
        else
          fat_gk_small_kernel<T, 1><<<n, 256, 0, s>>>(g, U, GV, GW, w, out, c);
        break;
    }
    return hipGetLastError();
  }
  const int nt = link_tiles(g);
  switch (stage) {
    case 0:
      fat_fk1_kernel<T><<<nt, kBlock, 0, s>>>(g, U, w, c, nt);
      break;
    case 1:
      fat_fk2_kernel<T><<<nt, kBlock, 0, s>>>(g, U, w, c, nt);
      break;
    case 2:
      fat_bk3_kernel<T><<<nt, kBlock, 0, s>>>(g, U, GV, w, nt);
      break;
    case 3:
      fat_bk2_kernel<T><<<nt, kBlock, 0, s>>>(g, U, GV, w, c, nt);
      break;
    default: {
      // two workgroups per CU (56 KiB LDS reservation, no LDS used): fewer links in
      // flight keep more of the gathered neighbour matrices in L2 (FP32 at 32^3 x 64:
      // 8.97 -> 8.54 ms; FP64 is at two per CU by registers anyway)
      const size_t lds = 56 * 1024;
      if (mode == 0)
        fat_gk_kernel<T, 0><<<nt, kBlock, lds, s>>>(g, U, GV, GW, w, out, c, nt);
      else
        fat_gk_kernel<T, 1><<<nt, kBlock, lds, s>>>(g, U, GV, GW, w, out, c, nt);
      break;
    }
  }
  return hipGetLastError();
}

#ifndef SYM_ONLY_F64
template hipError_t launch_fat_fk3<float>(const Geom&, const float*, float*, float*, const FatCoeffs&,
                                            const Fields<float>&, hipStream_t);
template hipError_t launch_fat_stage<float>(int, const Geom&, const float*, const float*, const float*, float*, int,
                                            const FatCoeffs&, const Fields<float>&, hipStream_t);
#endif
#ifndef SYM_ONLY_F32
template hipError_t launch_fat_fk3<double>(const Geom&, const double*, double*, double*, const FatCoeffs&,
                                             const Fields<double>&, hipStream_t);
template hipError_t launch_fat_stage<double>(int, const Geom&, const double*, const double*, const double*, double*,
                                             int, const FatCoeffs&, const Fields<double>&, hipStream_t);
#endif

}  // namespace sym
