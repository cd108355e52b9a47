// Wilson fermion force with clover term for given vectors X, Y: clover insertion kernel and
// the per-link force kernel.
//
// arXiv:1808.02281, Sec. "Wilson fermion action with clover term". With
// D = A - kappa Dh (eq. 18_7_17_2), hopping part of eq. 18_7_17_4 and clover diagonal
// A_n = 1 - c_sw kappa/16 sum_{mu != nu} [g_mu, g_nu] Q_{n;mu nu} (eq. 18_7_18_0; kappa =
// 1/(2(m+4))), the kernels differentiate Psi(U) = Y^+ D X + c.c. (eq. 18_6_24_0) along
// U_{k,rho} -> exp(i omega.T) U_{k,rho} and store G = -(1/2) M_TA with
// dPsi/domega^a = Re tr(i T_a M) = -2i tr(T_a G).
//
// Hopping (eqs. 18_1_29_20_1..3): with B' = sum_a ((1 - g_rho) X_{k+rho})_a (x) Y_{k,a}^+
// and C' = sum_a X_{k,a} (x) ((1 + g_rho) Y_{k+rho})_a^+ (colour outer products summed
// over spin a), B = U B' and C = C' U^+, and M_hop = -2 kappa (B - C). Both spin sums need
// only two terms, with both spinors projected (see outer).
//
// Clover: Y_n^+ G P X_n = tr(P S_n) for a colour matrix P with
// S_n = sum_a (G X_n)_a (x) Y_{n,a}^+, so the clover part of Psi is
// -(c_sw kappa / 8) Re sum_n sum_{mu<nu} tr(Q_{n;mu nu} K_n^{mu nu}), K = S - S^+ with
// G = [g_mu, g_nu]. Pass 1 (wilson_clover_kernel) stores the six K per site. The leaves
// through link (k, rho) lie in the plaquettes k -> k+rho -> k+rho+nu_s -> k+nu_s -> k
// (nu_s = +-nu), each a leaf of Q at its four corners c0..c3; splitting each leaf at
// U_{k,rho} (eqs. 18_7_26_9, 18_7_26_10, in matrix form) gives
//   M_clov = -(c_sw kappa / 8) U sum_{nu, s} sigma (abd K_c0 + K_c1 abd + a K_c2 bd + ab K_c3 d),
// with a = U_{k+rho,nu_s}, b = U_{k+rho+nu_s,-rho}, d = U_{k+nu_s,-nu_s}, and
// sigma = +-1 as the plaquette's sense rho -> nu_s agrees with the leaf sense min -> max.
// The last two terms share their outer factors, a (K_c2 b + b K_c3) d, and the first two have
// the same K for both signs s of nu, so they act on the sum over s: 14 products per (rho, nu)
// plane, 44 per link with U B' and C' U^+ (against 50 with each plaquette by itself: the
// FP32 pass issues a VALU instruction on every cycle, so it pays by the instruction).
//
// Spinor layout: field[p][3*spin + colour][V/2] complex (parity p, checkerboard cb).
// Clover insertions, pair = (0,1),(0,2),(0,3),(1,2),(1,3),(2,3): K is anti-Hermitian,
// so each is stored in 9 reals, block K[p][pair] of 9 V/2 reals = complex planes
// K01, K02, K12, (Im K00, Im K11), then a real plane Im K22; half the bytes of a full
// matrix on both sides (the force kernel reads 24 of them per link). Links are read as
// their first two rows, the third rebuilt (special unitary).
// Gamma matrices: Hermitian, DeGrand-Rossi basis, g_1..g_4 along x, y, z, t.
#include "kernels.hpp"

namespace sym {

namespace {

template <typename T>
struct spinor {
  cx<T> s[4][3];
};

template <typename T>
__device__ __forceinline__ cx<T> cmul(cx<T> a, cx<T> b) {
  return cx<T>{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename T>
__device__ __forceinline__ cx<T> times_i(cx<T> a, int sgn) {  // sgn * i * a
  return sgn > 0 ? cx<T>{-a.im, a.re} : cx<T>{a.im, -a.re};
}
template <typename T>
__device__ __forceinline__ cx<T> neg(cx<T> a) {
  return cx<T>{-a.re, -a.im};
}

// gamma_mu x (spin rows, per colour)
template <typename T>
__device__ __forceinline__ spinor<T> gamma_apply(int mu, const spinor<T>& x) {
  spinor<T> r;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (mu == 0) {
      r.s[0][c] = times_i(x.s[3][c], 1);
      r.s[1][c] = times_i(x.s[2][c], 1);
      r.s[2][c] = times_i(x.s[1][c], -1);
      r.s[3][c] = times_i(x.s[0][c], -1);
    } else if (mu == 1) {
      r.s[0][c] = neg(x.s[3][c]);
      r.s[1][c] = x.s[2][c];
      r.s[2][c] = x.s[1][c];
      r.s[3][c] = neg(x.s[0][c]);
    } else if (mu == 2) {
      r.s[0][c] = times_i(x.s[2][c], 1);
      r.s[1][c] = times_i(x.s[3][c], -1);
      r.s[2][c] = times_i(x.s[0][c], -1);
      r.s[3][c] = times_i(x.s[1][c], 1);
    } else {
      r.s[0][c] = x.s[2][c];
      r.s[1][c] = x.s[3][c];
      r.s[2][c] = x.s[0][c];
      r.s[3][c] = x.s[1][c];
    }
  }
  return r;
}

// sum over spin of the colour outer product: out_{ba} = sum_alpha p_{alpha b} conj(q_{alpha a})
template <typename T>
__device__ __forceinline__ su3<T> outer(const spinor<T>& p, const spinor<T>& q) {
  su3<T> r;
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      T re = T(0), im = T(0);
#pragma unroll
      for (int al = 0; al < 4; ++al) {
        const cx<T> x = p.s[al][b], y = q.s[al][a];
        re = fma(x.re, y.re, re);
        re = fma(x.im, y.im, re);
        im = fma(x.im, y.re, im);
        im = fma(-x.re, y.im, im);
      }
      r.e[3 * b + a] = cx<T>{re, im};
    }
  return r;
}

template <typename T>
__device__ __forceinline__ spinor<T> load_spinor(const T* F, int p, int Vh, int cb) {
  const cx<T>* blk = reinterpret_cast<const cx<T>*>(F) + (size_t)p * 12 * (size_t)Vh;
  const unsigned bytes = 12u * (unsigned)Vh * (unsigned)sizeof(cx<T>);
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<cx<T>*>(blk), (short)0, (int)bytes,
                                                                     kBufferWord3);
  const int voff = cb * (int)sizeof(cx<T>);
  spinor<T> s;
#pragma unroll
  for (int e = 0; e < 12; ++e) {
    const int soff = (int)((unsigned)e * (unsigned)Vh * (unsigned)sizeof(cx<T>));
    if constexpr (sizeof(T) == 4)
      s.s[e / 3][e % 3] = __builtin_bit_cast(cx<T>, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    else
      s.s[e / 3][e % 3] = __builtin_bit_cast(cx<T>, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
  }
  return s;
}

// Spin components 0 and 1 of (1 + sgn gamma_rho) x at a site. They carry the whole
// projection: component a is paired with b(a) by the one non-zero of row a of gamma_rho,
// (1 + sgn gamma_rho) x is x_a + sgn phase_a x_{b(a)} there, and its components 2 and 3 are
// phases times these two. rho is wave-uniform.
template <typename T>
struct half_spinor {
  cx<T> s[2][3];
};

template <typename T>
__device__ __forceinline__ half_spinor<T> load_projected(const T* F, int p, int Vh, int cb, int rho, T sgn) {
  const cx<T>* blk = reinterpret_cast<const cx<T>*>(F) + (size_t)p * 12 * (size_t)Vh;
  const unsigned bytes = 12u * (unsigned)Vh * (unsigned)sizeof(cx<T>);
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<cx<T>*>(blk), (short)0, (int)bytes,
                                                                     kBufferWord3);
  const int voff = cb * (int)sizeof(cx<T>);
  const bool imag = rho == 0 || rho == 2;
  half_spinor<T> h;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int b = rho < 2 ? 3 - a : 2 + a;
    const T sg = (rho == 1 && a == 0) || (rho == 2 && a == 1) ? -sgn : sgn;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      cx<T> v[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int soff = (int)((unsigned)(3 * (k ? b : a) + c) * (unsigned)Vh * (unsigned)sizeof(cx<T>));
        if constexpr (sizeof(T) == 4)
          v[k] = __builtin_bit_cast(cx<T>, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
        else
          v[k] = __builtin_bit_cast(cx<T>, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
      }
      const T re = imag ? -v[1].im : v[1].re, im = imag ? v[1].re : v[1].im;
      h.s[a][c] = cx<T>{fma(sg, re, v[0].re), fma(sg, im, v[0].im)};
    }
  }
  return h;
}

// Colour outer product of two spinors projected with the same (1 +- gamma_rho) = 2 P:
// sum over all four spins of (2P x)_b conj(y_a) = sum over two of (2P x)_b conj((2P y)_a),
// since P is a Hermitian projector and the lower components repeat the upper ones.
template <typename T>
__device__ __forceinline__ su3<T> outer(const half_spinor<T>& p, const half_spinor<T>& q) {
  su3<T> r;
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      T re = T(0), im = T(0);
#pragma unroll
      for (int al = 0; al < 2; ++al) {
        const cx<T> x = p.s[al][b], y = q.s[al][a];
        re = fma(x.re, y.re, re);
        re = fma(x.im, y.im, re);
        im = fma(x.im, y.re, im);
        im = fma(-x.re, y.im, im);
      }
      r.e[3 * b + a] = cx<T>{re, im};
    }
  return r;
}

constexpr int pair_index(int lo, int hi) { return lo == 0 ? hi - 1 : (lo == 1 ? hi + 1 : 5); }

template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t antiherm_rsrc(const T* blk, int Vh) {
  const unsigned bytes = 9u * (unsigned)Vh * (unsigned)sizeof(T);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(blk), (short)0, (int)bytes, kBufferWord3);
}

// the anti-Hermitian k into its 9-real block (layout above)
template <typename T>
__device__ __forceinline__ void store_antiherm(T* blk, int Vh, int cb, const su3<T>& k) {
  const __amdgpu_buffer_rsrc_t r = antiherm_rsrc(static_cast<const T*>(blk), Vh);
  const cx<T> v[4] = {k.e[1], k.e[2], k.e[5], cx<T>{k.e[0].im, k.e[4].im}};
  const int voff = cb * (int)sizeof(cx<T>);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int soff = (int)((unsigned)c * (unsigned)Vh * (unsigned)sizeof(cx<T>));
    if constexpr (sizeof(T) == 4)
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(__attribute__((ext_vector_type(2))) unsigned, v[c]),
                                            r, voff, soff, kStoreNT);
    else
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, v[c]),
                                             r, voff, soff, kStoreNT);
  }
  const int voff1 = cb * (int)sizeof(T), soff1 = (int)(8u * (unsigned)Vh * (unsigned)sizeof(T));
  if constexpr (sizeof(T) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, k.e[8].im), r, voff1, soff1, kStoreNT);
  else
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(__attribute__((ext_vector_type(2))) unsigned, k.e[8].im),
                                          r, voff1, soff1, kStoreNT);
}

template <typename T>
__device__ __forceinline__ su3<T> load_antiherm(const T* blk, int Vh, int cb) {
  const __amdgpu_buffer_rsrc_t r = antiherm_rsrc(blk, Vh);
  const int voff = cb * (int)sizeof(cx<T>);
  cx<T> v[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int soff = (int)((unsigned)c * (unsigned)Vh * (unsigned)sizeof(cx<T>));
    if constexpr (sizeof(T) == 4)
      v[c] = __builtin_bit_cast(cx<T>, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    else
      v[c] = __builtin_bit_cast(cx<T>, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
  }
  const int voff1 = cb * (int)sizeof(T), soff1 = (int)(8u * (unsigned)Vh * (unsigned)sizeof(T));
  T d2;
  if constexpr (sizeof(T) == 4)
    d2 = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff1, soff1, 0));
  else
    d2 = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, voff1, soff1, 0));
  su3<T> k;
  k.e[0] = cx<T>{T(0), v[3].re};
  k.e[1] = v[0];
  k.e[2] = v[1];
  k.e[3] = cx<T>{-v[0].re, v[0].im};
  k.e[4] = cx<T>{T(0), v[3].im};
  k.e[5] = v[2];
  k.e[6] = cx<T>{-v[1].re, v[1].im};
  k.e[7] = cx<T>{-v[2].re, v[2].im};
  k.e[8] = cx<T>{T(0), d2};
  return k;
}

// pass 1: K^{mu nu} = S - S^+, S = sum_a ([g_mu, g_nu] X)_a (x) Y_a^+, for every site
template <typename T>
__global__ __launch_bounds__(kBlock) void wilson_clover_kernel(Geom g, const T* __restrict__ X,
                                                                const T* __restrict__ Y, T* __restrict__ K) {
  const long long idx = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (idx >= 2ll * g.Vh) return;
  const int p = (int)(idx / g.Vh), cb = (int)(idx - (long long)p * g.Vh);
  const spinor<T> x = load_spinor(X, p, g.Vh, cb);
  const spinor<T> y = load_spinor(Y, p, g.Vh, cb);
  spinor<T> gx[4];
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) gx[mu] = gamma_apply(mu, x);
#pragma unroll
  for (int mu = 0; mu < 4; ++mu)
#pragma unroll
    for (int nu = mu + 1; nu < 4; ++nu) {
      const spinor<T> a = gamma_apply(mu, gx[nu]), b = gamma_apply(nu, gx[mu]);
      spinor<T> cm;
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) cm.s[s][c] = cx<T>{a.s[s][c].re - b.s[s][c].re, a.s[s][c].im - b.s[s][c].im};
      const su3<T> S = outer(cm, y);
      su3<T> k;
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const cx<T> sij = S.e[3 * i + j], sji = S.e[3 * j + i];
          k.e[3 * i + j] = cx<T>{sij.re - sji.re, sij.im + sji.im};
        }
      store_antiherm(K + (size_t)((p * 6 + pair_index(mu, nu)) * 9) * (size_t)g.Vh, g.Vh, cb, k);
    }
}

template <typename T>
struct WCtx {
  const T* U;
  const T* K;
  int Vh;
  int p;
  int ax[4];
  Nbr nb;

  template <int D0, int D1, int D2, int D3, int A>
  __device__ __forceinline__ su3<T> u() const {
    constexpr int dp = offset_parity<D0, D1, D2, D3>();
    return load_su3_rows(block_ptr(U, ax[A], p ^ dp, Vh), Vh, nbr_cb<D0, D1, D2, D3>(nb));
  }
  template <int D0, int D1, int D2, int D3>
  __device__ __forceinline__ su3<T> k(int pair) const {
    constexpr int dp = offset_parity<D0, D1, D2, D3>();
    return load_antiherm(K + (size_t)((((p ^ dp) * 6) + pair) * 9) * (size_t)Vh, Vh, nbr_cb<D0, D1, D2, D3>(nb));
  }
};

template <typename T>
__device__ __forceinline__ su3<T> dagger(const su3<T>& a) {
  su3<T> r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) r.e[3 * i + j] = cx<T>{a.e[3 * j + i].re, -a.e[3 * j + i].im};
  return r;
}

// Products with an insertion K, whose diagonal is imaginary: its zero real parts are left out
// (the compiler keeps a multiplication by a constant zero), 90 instructions against 108.
//   add_k<false, D>: C += K M^{D};  add_k<true, D>: C += M^{D} K;  with SET, C is set instead.
template <bool RIGHT, bool D, bool SET, typename T>
__device__ __forceinline__ void add_k(su3<T>& c, const su3<T>& k, const su3<T>& m) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      T re = SET ? T(0) : c.e[3 * i + j].re, im = SET ? T(0) : c.e[3 * i + j].im;
      bool fresh = SET;
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        const cx<T> x = RIGHT ? elem<D>(m, i, l) : k.e[3 * i + l];
        const cx<T> y = RIGHT ? k.e[3 * l + j] : elem<D>(m, l, j);
        if (RIGHT ? l == j : l == i) {  // the imaginary diagonal: x.re (or y.re) is zero
          const T a = RIGHT ? y.im : x.im;
          const cx<T> b = RIGHT ? x : y;
          re = fresh ? -a * b.im : fma(-a, b.im, re);
          im = fresh ? a * b.re : fma(a, b.re, im);
        } else {
          re = fresh ? x.re * y.re : fma(x.re, y.re, re);
          im = fresh ? x.re * y.im : fma(x.re, y.im, im);
          re = fma(-x.im, y.im, re);
          im = fma(x.im, y.re, im);
        }
        fresh = false;
      }
      c.e[3 * i + j] = cx<T>{re, im};
    }
}

// C -= A B
template <typename T>
__device__ __forceinline__ void mac_neg(su3<T>& c, const su3<T>& a, const su3<T>& b) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      T re = c.e[3 * i + j].re, im = c.e[3 * i + j].im;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const cx<T> x = a.e[3 * i + k], y = b.e[3 * k + j];
        re = fma(-x.re, y.re, re);
        im = fma(-x.re, y.im, im);
        re = fma(x.im, y.im, re);
        im = fma(-x.im, y.re, im);
      }
      c.e[3 * i + j] = cx<T>{re, im};
    }
}

// The plaquette k, k+rho, k+rho+nu_s, k+nu_s with nu = ax[J], s = S: abd into w and
// a (K2 b + b K3) d into t, both set for S > 0 and subtracted for S < 0.
template <int J, int S, typename T>
__device__ __forceinline__ void clover_plaquette(su3<T>& t, su3<T>& w, const WCtx<T>& c0) {
  WCtx<T> c = c0;
  asm volatile("" : "+s"(c.U), "+s"(c.K));
  constexpr int e1 = J == 1 ? 1 : 0, e2 = J == 2 ? 1 : 0, e3 = J == 3 ? 1 : 0;
  constexpr int f1 = S * e1, f2 = S * e2, f3 = S * e3;
  const int rho = c.ax[0], nu = c.ax[J];
  const int pair = rho < nu ? pair_index(rho, nu) : pair_index(nu, rho);
  su3<T> ab, ax;
  {
    const su3<T> ub = c.template u<0, f1, f2, f3, 0>();  // b = ub^dagger
    su3<T> x;  // K2 b + b K3
    add_k<false, true, true>(x, c.template k<1, f1, f2, f3>(pair), ub);
    add_k<true, true, false>(x, c.template k<0, f1, f2, f3>(pair), ub);
    su3<T> a;
    if constexpr (S > 0)
      a = c.template u<1, 0, 0, 0, J>();
    else
      a = dagger(c.template u<1, -e1, -e2, -e3, J>());
    ab = mul<false, true>(a, ub);
    ax = mul<false, false>(a, x);
  }
  __builtin_amdgcn_sched_barrier(0);
  su3<T> d;
  if constexpr (S > 0)
    d = dagger(c.template u<0, 0, 0, 0, J>());
  else
    d = c.template u<0, -e1, -e2, -e3, J>();
  if constexpr (S > 0) {
    w = mul<false, false>(ab, d);
    t = mul<false, false>(ax, d);
  } else {
    mac_neg(w, ab, d);
    mac_neg(t, ax, d);
  }
}

// acc += sum over s of sigma (abd K0 + K1 abd + a K2 bd + ab K3 d) for the two plaquettes in
// the (rho, nu) plane, nu = ax[J], sigma = s (rho < nu ? 1 : -1). Both have the insertions
// K0, K1 of the link's own ends, so these act once on the difference w of the two abd. The
// plane is summed by itself before it is added to acc (in FP32 the error against 64 bits is
// then no larger than with each plaquette summed by itself).
template <int J, typename T>
__device__ __forceinline__ void clover_plane(su3<T>& acc, const WCtx<T>& c0) {
  su3<T> t, w;
  clover_plaquette<J, 1>(t, w, c0);
  __builtin_amdgcn_sched_barrier(0);
  clover_plaquette<J, -1>(t, w, c0);
  __builtin_amdgcn_sched_barrier(0);
  WCtx<T> c = c0;
  asm volatile("" : "+s"(c.U), "+s"(c.K));
  const int rho = c.ax[0], nu = c.ax[J];
  const int pair = rho < nu ? pair_index(rho, nu) : pair_index(nu, rho);
  add_k<true, false, false>(t, c.template k<0, 0, 0, 0>(pair), w);
  add_k<false, false, false>(t, c.template k<1, 0, 0, 0>(pair), w);
  axpy(acc, T(rho < nu ? 1 : -1), t);
  __builtin_amdgcn_sched_barrier(0);
}

template <typename T>
__device__ __forceinline__ WCtx<T> make_wctx(const Geom& g, const T* U, const T* K, int mu, int p, int cb) {
  WCtx<T> c;
  int x[4];
  cb_coords(g, p, cb, x);
  c.U = U;
  c.K = K;
  c.Vh = g.Vh;
  c.p = p;
  c.ax[0] = mu;
  c.ax[1] = mu == 0 ? 1 : 0;
  c.ax[2] = mu <= 1 ? 2 : 1;
  c.ax[3] = mu <= 2 ? 3 : 2;
  Nbr full;
  make_nbr(g, x, full);
#pragma unroll
  for (int fa = 0; fa < 4; ++fa) {
    const int a = c.ax[fa];
#pragma unroll
    for (int dd = 0; dd < 5; ++dd)
      c.nb.o[fa][dd] = a == 0 ? full.o[0][dd] : a == 1 ? full.o[1][dd] : a == 2 ? full.o[2][dd] : full.o[3][dd];
  }
  return c;
}

// The hopping outer products B' and C' of the link.
template <typename T>
__device__ __forceinline__ su3<T> hop_b(const WCtx<T>& c, const T* X, const T* Y, int cb) {
  return outer(load_projected(X, c.p ^ 1, c.Vh, nbr_cb<1, 0, 0, 0>(c.nb), c.ax[0], T(-1)),
               load_projected(Y, c.p, c.Vh, cb, c.ax[0], T(-1)));
}
template <typename T>
__device__ __forceinline__ su3<T> hop_c(const WCtx<T>& c, const T* X, const T* Y, int cb) {
  return outer(load_projected(X, c.p, c.Vh, cb, c.ax[0], T(1)),
               load_projected(Y, c.p ^ 1, c.Vh, nbr_cb<1, 0, 0, 0>(c.nb), c.ax[0], T(1)));
}

// M = U (-2 kappa B' + w acc) + 2 kappa C' U^+, w = -c_sw kappa / 8: the inner factor, and the
// result from M's two terms.
template <typename T>
__device__ __forceinline__ su3<T> wilson_inner(const su3<T>& Bp, const su3<T>& acc, double kappa, double csw) {
  const T w = T(-csw * kappa / 8.0), mk = T(-2.0 * kappa);
  su3<T> inner;
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    inner.e[e].re = fma(mk, Bp.e[e].re, w * acc.e[e].re);
    inner.e[e].im = fma(mk, Bp.e[e].im, w * acc.e[e].im);
  }
  return inner;
}
template <typename T>
__device__ __forceinline__ void store_wilson(const WCtx<T>& c, T* out, int cb, const su3<T>& u, const su3<T>& inner,
                                             const su3<T>& cu, double kappa) {
  su3<T> M = mul<false, false>(u, inner);
  axpy(M, T(2.0 * kappa), cu);
  store_link(block_ptr(out, c.ax[0], c.p, c.Vh), c.Vh, cb, ta_scaled(M, T(-0.5)));
}

// FP32: two waves per SIMD (199 VGPRs); three would spill: 1.75 against 1.50 ms at
// 32^3 x 64. FP64: one wave (256 VGPRs and 162 AGPRs). With one sum over s per plane,
// projected spinors and the insertions' zero parts left out, FP32 1.63 -> 1.46 ms at 32^3 x 64,
// FP64 1.05 -> 0.96 ms at 24^3 x 48. Where a lattice has 2,049 to 3,072 waves, which take two rounds
// at two waves per SIMD and took one at three, FP32 gains nothing: 14 x 12 x 14^2 43.2 -> 43.0 us a call,
// 16 x 12 x 14^2 41.8 -> 42.1, 14^4 43.4 -> 43.5, 16^3 x 12 45.1 -> 43.6. (abd as two rows with the third
// rebuilt would save another 2%, at an error against 64 bits that is no longer below that of
// the separate plaquettes.)
template <typename T>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 2 : 1))) void
wilson_force_kernel(Geom g, const T* __restrict__ U, const T* __restrict__ X, const T* __restrict__ Y,
                    const T* __restrict__ K, T* __restrict__ out, double kappa, double csw, int ntiles) {
  const LinkTile lt = link_tile(g, blockIdx.x, ntiles);
  const int cb = lt.chunk * kBlock + threadIdx.x;
  if (cb >= g.Vh) return;
  const WCtx<T> c = make_wctx(g, U, K, lt.mu, lt.p, cb);

  // clover leaves through the link
  su3<T> acc;
  set_zero(acc);
  if (csw != 0.0) {
    clover_plane<1>(acc, c);
    clover_plane<2>(acc, c);
    clover_plane<3>(acc, c);
  }
  const su3<T> inner = wilson_inner(hop_b(c, X, Y, cb), acc, kappa, csw);
  __builtin_amdgcn_sched_barrier(0);
  const su3<T> Cp = hop_c(c, X, Y, cb);
  const su3<T> u = c.template u<0, 0, 0, 0, 0>();
  store_wilson(c, out, cb, u, inner, mul<false, true>(Cp, u), kappa);
}

// Small lattices: four waves share 64 links (one per lane of every wave), waves 0..2 the
// clover leaves of a plane each, wave 3 the hopping terms, joined in LDS. With a wave per 64
// links the clover term is a serial stream of 5,500 instructions whatever the lattice. The
// same operations in the same order: bitwise the same force. It pays up to two workgroups per CU:
// kernel 4^4 FP32 20 -> 9 us, FP64 21 -> 11 us; 8^3 x 16 (512 workgroups) 22 -> 13 and 26 -> 21 us.
// Above, FP64 loses (8^3 x 18, 576: 24.3 -> 27.7 us; 1,024: 27.4 -> 37.9) and FP32 gains little (576 to
// 768: 20 -> 17.5 us) or loses (1,024: 21.3 either way; 12^4, 1,296: 25.9 -> 27.3).
template <typename T>
__global__ __launch_bounds__(256) void wilson_force_small_kernel(Geom g, const T* __restrict__ U,
                                                                 const T* __restrict__ X, const T* __restrict__ Y,
                                                                 const T* __restrict__ K, T* __restrict__ out,
                                                                 double kappa, double csw) {
  __shared__ T lds[4 * 18 * 64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const LdsMats<T> m{lds, (int)(threadIdx.x & 63)};
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const bool active = (tile >> 3) * 64 + m.lane < g.Vh;
  const int cb = active ? (tile >> 3) * 64 + m.lane : 0;
  const WCtx<T> c = make_wctx(g, U, K, tile & 3, (tile >> 2) & 1, cb);
  su3<T> acc;
  set_zero(acc);
  if (active) {
    if (wave == 0) {
      clover_plane<1>(acc, c);
    } else if (wave == 1) {
      clover_plane<2>(acc, c);
      m.put(0, acc);
    } else if (wave == 2) {
      clover_plane<3>(acc, c);
      m.put(1, acc);
    } else {
      m.put(2, hop_b(c, X, Y, cb));
      m.put(3, mul<false, true>(hop_c(c, X, Y, cb), c.template u<0, 0, 0, 0, 0>()));
    }
  }
  __syncthreads();
  if (!active || wave != 0) return;
  add(acc, m.get(0));
  add(acc, m.get(1));
  store_wilson(c, out, cb, c.template u<0, 0, 0, 0, 0>(), wilson_inner(m.get(2), acc, kappa, csw), m.get(3), kappa);
}

}  // namespace

template <typename T>
hipError_t launch_wilson_clover(const Geom& g, const T* X, const T* Y, T* K, hipStream_t s) {
  const long long n = 2ll * g.Vh;
  wilson_clover_kernel<T><<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(g, X, Y, K);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_wilson_force(const Geom& g, const T* U, const T* X, const T* Y, const T* K, T* out, double kappa,
                               double csw, hipStream_t s) {
  if (csw != 0.0 && link_tiles(g, 64) <= 2 * kCUs) {
    wilson_force_small_kernel<T><<<link_tiles(g, 64), 256, 0, s>>>(g, U, X, Y, K, out, kappa, csw);
    return hipGetLastError();
  }
  const int nt = link_tiles(g);
  wilson_force_kernel<T><<<nt, kBlock, 0, s>>>(g, U, X, Y, K, out, kappa, csw, nt);
  return hipGetLastError();
}

#ifndef SYM_ONLY_F64
template hipError_t launch_wilson_clover<float>(const Geom&, const float*, const float*, float*, hipStream_t);
template hipError_t launch_wilson_force<float>(const Geom&, const float*, const float*, const float*, const float*,
                                               float*, double, double, hipStream_t);
#endif
#ifndef SYM_ONLY_F32
template hipError_t launch_wilson_clover<double>(const Geom&, const double*, const double*, double*, hipStream_t);
template hipError_t launch_wilson_force<double>(const Geom&, const double*, const double*, const double*,
                                                const double*, double*, double, double, hipStream_t);
#endif

}  // namespace sym
