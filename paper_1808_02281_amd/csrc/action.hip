// Symanzik action S_G (arXiv:1808.02281 Sec. II, eq. 18_6_4_1) and the final
// deterministic reductions shared by the action, the fused force action and the
// leapfrog Hamiltonian.
//
// Action kernel: w_X = sum over sites and class-X loops of (3 - Re tr P), in double, with
// the 34 loops of a site (eq. 18_6_6_3_0), the last product of each replaced by its trace.
// No unitarity is assumed, so the links are read in full.
//
// A workgroup is 64 sites whose four waves share the loops. With one thread per site, what
// bounded the kernel was link data from beyond the L2 (16 GB for 0.4 GB of links at 24^3 x 48
// in FP64, 7.1 TB/s). 64 sites per workgroup instead of 256 keep the links of the sites in
// flight on an XCD within its 4 MiB of L2 (1.5 GB fetched), in the t-fastest slab order of the
// other passes, and small lattices get four times the waves with a quarter of the serial work
// each. The axes are wave-uniform values rather than template arguments, so the four waves
// share one code. The bound now is the vector load path (TD busy 0.94 in FP64, VALU 0.44): 140
// matrices are loaded per site (FP32 160), half of them L1 hits and most of the rest L2 hits.
//
// FP32 multiplies every loop out from its base site link by link (loops that start with the
// same two links share that product): the double sums carry the float rounding of every
// trace, and this way an FP32 action does not depend on how the loops are shared. FP64
// closes the loops from halves that meet in a trace, fewer loads for the same products. With the
// two ways around the (nu, rho) square of a site, P = U_{y,nu} U_{y+nu,rho} and
// Q = U_{y,rho} U_{y+rho,nu}:
//   plaquette   tr(P Q^+);
//   rectangles  tr((U_{y,nu} P_{y+nu}) (Q_y U_{y+nu+rho,nu})^+) and the same with nu and
//               rho exchanged;
//   cube loops  carry one side of the square along mu: (mu, nu, rho, -mu, -nu, -rho) is
//               tr((U_{y,mu} P_{y+mu}) (Q_y U_{y+nu+rho,mu})^+), exchanging P and Q gives the
//               loop with nu and rho both reversed, and the two loops with one of them
//               reversed have the same form with the square's other two sides
//               E = U_{y+rho,nu} U_{y+nu,rho}^+ and F = U_{y,rho}^+ U_{y,nu}.
// Every loop is summed once over the lattice (its base site differs by a translation). Four
// (square, mu) pairs cover the four axis triples.
//
// Measured, before -> now: FP64 24^3 x 48 2.25 -> 0.61 ms (0.74 ms with the FP32 form), 4^4
// 107 -> 17 us; FP32 32^3 x 64 3.37 -> 1.38 ms (halves: 1.08 to 1.21 ms).
#include "kernels.hpp"

namespace sym {
namespace {

// Lexicographic index steps of one and two links forwards and one backwards along an axis.
struct Step {
  int one, two, back;
};

template <typename T>
struct LoopSite {
  const T* U;
  int Vh;
  int p;
  int lex;

  // U_{y+d, a} for the site y + d at lexicographic step `off` and parity flip k
  __device__ __forceinline__ su3<T> link(int a, int k, int off) const {
    return load_link(block_ptr(U, a, p ^ k, Vh), Vh, (lex + off) >> 1);
  }
};

// Fence between loops: links that several loops read are loaded again (they hit L1) rather
// than kept in registers, no load moves ahead of its loop, and the loop's sum is finished
// where it stands (the compiler otherwise sinks the products to the use of w and keeps
// every link alive until there).
template <typename T>
__device__ __forceinline__ LoopSite<T> next_loop(const LoopSite<T>& s, double& w) {
  LoopSite<T> r = s;
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" : "+s"(r.U), "+v"(w));
  return r;
}

__device__ __forceinline__ Step step_along(const Geom& g, const int x[4], int a) {
  const int xa = a == 0 ? x[0] : a == 1 ? x[1] : a == 2 ? x[2] : x[3];
  const int La = a == 0 ? g.L[0] : a == 1 ? g.L[1] : a == 2 ? g.L[2] : g.L[3];
  const int stride = a == 0 ? 1 : a == 1 ? g.L[0] : a == 2 ? g.L[0] * g.L[1] : g.L[0] * g.L[1] * g.L[2];
  Step s;
  s.one = (xa + 1 < La ? 1 : 1 - La) * stride;
  s.two = (xa + 2 < La ? 2 : 2 - La) * stride;
  s.back = (xa > 0 ? -1 : La - 1) * stride;
  return s;
}

// ----------------------------------------------------------- loop by loop (FP32)

// (m, n, -m, -n)
template <typename T>
__device__ __forceinline__ void plaquette(const LoopSite<T>& s0, int m, int n, Step dm, Step dn, double& w) {
  const LoopSite<T> s = next_loop(s0, w);
  su3<T> p = mul<false, false>(s.link(m, 0, 0), s.link(n, 1, dm.one));
  p = mul<false, true>(p, s.link(m, 1, dn.one));
  w += 3.0 - re_tr_mul<true>(p, s.link(n, 0, 0));
}

// (m, m, n, -m, -m, -n), mm = U_{x,m} U_{x+m,m}
template <typename T>
__device__ __forceinline__ void rectangle(const LoopSite<T>& s0, const su3<T>& mm, int m, int n, Step dm, Step dn,
                                          double& w) {
  const LoopSite<T> s = next_loop(s0, w);
  su3<T> p = mul<false, false>(mm, s.link(n, 0, dm.two));
  p = mul<false, true>(p, s.link(m, 0, dm.one + dn.one));
  p = mul<false, true>(p, s.link(m, 1, dn.one));
  w += 3.0 - re_tr_mul<true>(p, s.link(n, 0, 0));
}

// (m, SN n, SR r, -m, -SN n, -SR r), mn = U_{x,m} U_{x+m,SN n}
template <int SN, int SR, typename T>
__device__ __forceinline__ void cube_loop(const LoopSite<T>& s0, const su3<T>& mn, int m, int n, int r, Step dm,
                                          Step dn, Step dr, double& w) {
  const LoopSite<T> s = next_loop(s0, w);
  const int on = SN > 0 ? dn.one : dn.back, orr = SR > 0 ? dr.one : dr.back;
  su3<T> p;
  if constexpr (SR > 0)
    p = mul<false, false>(mn, s.link(r, 0, dm.one + on));
  else
    p = mul<false, true>(mn, s.link(r, 1, dm.one + on + dr.back));
  p = mul<false, true>(p, s.link(m, 0, on + orr));
  if constexpr (SN > 0)
    p = mul<false, true>(p, s.link(n, 1, orr));
  else
    p = mul<false, false>(p, s.link(n, 0, dn.back + orr));
  if constexpr (SR > 0)
    w += 3.0 - re_tr_mul<true>(p, s.link(r, 0, 0));
  else
    w += 3.0 - re_tr_mul<false>(p, s.link(r, 1, dr.back));
}

template <int SN, typename T>
__device__ __forceinline__ void cube_pair(const LoopSite<T>& s0, int m, int n, int r, Step dm, Step dn, Step dr,
                                          double& w) {
  const LoopSite<T> s = next_loop(s0, w);
  su3<T> mn;
  if constexpr (SN > 0)
    mn = mul<false, false>(s.link(m, 0, 0), s.link(n, 1, dm.one));
  else
    mn = mul<false, true>(s.link(m, 0, 0), s.link(n, 0, dm.one + dn.back));
  cube_loop<SN, 1>(s, mn, m, n, r, dm, dn, dr, w);
  cube_loop<SN, -1>(s, mn, m, n, r, dm, dn, dr, w);
}

// ------------------------------------------------------------------ halves (FP64)

// Plaquette and both rectangles of the (nu, rho) square: 8 products, 3 traces.
template <typename T>
__device__ __forceinline__ void square_loops(const LoopSite<T>& s0, int nu, int rho, Step dn, Step dr, double w[3]) {
  const LoopSite<T> s1 = next_loop(s0, w[1]);
  const su3<T> un = s1.link(nu, 0, 0), ur = s1.link(rho, 0, 0);
  const su3<T> P = mul<false, false>(un, s1.link(rho, 1, dn.one));
  const su3<T> Q = mul<false, false>(ur, s1.link(nu, 1, dr.one));
  w[0] += 3.0 - re_tr_mul<true>(P, Q);
  {  // long side along nu
    const LoopSite<T> s = next_loop(s1, w[0]);
    const su3<T> a = mul<false, false>(un, mul<false, false>(s.link(nu, 1, dn.one), s.link(rho, 0, dn.two)));
    const su3<T> b = mul<false, false>(Q, s.link(nu, 0, dn.one + dr.one));
    w[1] += 3.0 - re_tr_mul<true>(a, b);
  }
  {  // long side along rho
    const LoopSite<T> s = next_loop(s1, w[1]);
    const su3<T> a = mul<false, false>(ur, mul<false, false>(s.link(rho, 1, dr.one), s.link(nu, 0, dr.two)));
    const su3<T> b = mul<false, false>(P, s.link(rho, 0, dn.one + dr.one));
    w[1] += 3.0 - re_tr_mul<true>(a, b);
  }
  (void)next_loop(s1, w[1]);
}

// The four cube loops of the (nu, rho) square carried along mu: 16 products, 4 traces, the
// two diagonals of the square in turn (two waves per SIMD; the square's four sides at once
// would load 14 links instead of 20 but take 298 registers: 0.70 ms at one wave, 0.80 ms with
// spills at two, against 0.61).
template <typename T>
__device__ __forceinline__ void cube_loops(const LoopSite<T>& s0, int nu, int rho, int mu, Step dn, Step dr, Step dm,
                                           double w[3]) {
  {
    const LoopSite<T> s = next_loop(s0, w[2]);
    const su3<T> um = s.link(mu, 0, dn.one + dr.one);
    const su3<T> P = mul<false, false>(mul<false, false>(s.link(nu, 0, 0), s.link(rho, 1, dn.one)), um);
    const su3<T> Q = mul<false, false>(mul<false, false>(s.link(rho, 0, 0), s.link(nu, 1, dr.one)), um);
    __builtin_amdgcn_sched_barrier(0);
    const su3<T> u0 = s.link(mu, 0, 0);
    const su3<T> P1 = mul<false, false>(s.link(nu, 1, dm.one), s.link(rho, 0, dn.one + dm.one));
    w[2] += 3.0 - re_tr_mul<true>(mul<false, false>(u0, P1), Q);
    __builtin_amdgcn_sched_barrier(0);
    const su3<T> Q1 = mul<false, false>(s.link(rho, 1, dm.one), s.link(nu, 0, dr.one + dm.one));
    w[2] += 3.0 - re_tr_mul<true>(mul<false, false>(u0, Q1), P);
  }
  {
    const LoopSite<T> s = next_loop(s0, w[2]);
    const su3<T> um = s.link(mu, 1, dn.one);
    const su3<T> E = mul<false, false>(mul<false, true>(s.link(nu, 1, dr.one), s.link(rho, 1, dn.one)), um);
    const su3<T> F = mul<false, false>(mul<true, false>(s.link(rho, 0, 0), s.link(nu, 0, 0)), um);
    __builtin_amdgcn_sched_barrier(0);
    const su3<T> u1 = s.link(mu, 1, dr.one);
    const su3<T> E1 = mul<false, true>(s.link(nu, 0, dr.one + dm.one), s.link(rho, 0, dn.one + dm.one));
    w[2] += 3.0 - re_tr_mul<true>(mul<false, false>(u1, E1), F);
    __builtin_amdgcn_sched_barrier(0);
    const su3<T> F1 = mul<true, false>(s.link(rho, 1, dm.one), s.link(nu, 1, dm.one));
    w[2] += 3.0 - re_tr_mul<true>(mul<false, false>(u1, F1), E);
  }
  (void)next_loop(s0, w[2]);
}

constexpr int kActionSites = 64;  // sites per workgroup, one per lane of each of its waves

template <typename T>
__global__ __launch_bounds__(kBlock) void action_kernel(Geom g, const T* __restrict__ U, double* __restrict__ partials,
                                                        int ntiles) {
  const SiteTile st = site_tile(g, blockIdx.x, ntiles, kBlock / kActionSites);
  const int cb = st.chunk * kActionSites + (threadIdx.x & 63);
  double w[3] = {0.0, 0.0, 0.0};
  if (cb < g.Vh) {
    int x[4];
    cb_coords(g, st.p, cb, x);
    LoopSite<T> s;
    s.U = U;
    s.Vh = g.Vh;
    s.p = st.p;
    s.lex = 2 * cb + (x[0] & 1);
    // the waves' shares rotate with the workgroup, so that the longer ones do not always land
    // on the same SIMDs
    const int k = (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + (int)blockIdx.x) & 3;
    if constexpr (sizeof(T) == 4) {
      {  // cube loops of the triples 012, 013, 023, 123
        const int m = k == 3 ? 1 : 0, n = k < 2 ? 1 : 2, r = k == 0 ? 2 : 3;
        const Step dm = step_along(g, x, m), dn = step_along(g, x, n), dr = step_along(g, x, r);
        cube_pair<1>(s, m, n, r, dm, dn, dr, w[2]);
        cube_pair<-1>(s, m, n, r, dm, dn, dr, w[2]);
      }
      const Step dk = step_along(g, x, k);
      {  // rectangles with the long side along k
        const LoopSite<T> t = next_loop(s, w[2]);
        const su3<T> kk = mul<false, false>(t.link(k, 0, 0), t.link(k, 1, dk.one));
        const int a = k == 0 ? 1 : 0, b = k <= 1 ? 2 : 1, c = k <= 2 ? 3 : 2;
        rectangle(t, kk, k, a, dk, step_along(g, x, a), w[1]);
        rectangle(t, kk, k, b, dk, step_along(g, x, b), w[1]);
        rectangle(t, kk, k, c, dk, step_along(g, x, c), w[1]);
      }
      // plaquettes 01 03 | 12 13 | 23 | 02
      if (k < 3) plaquette(s, k, k + 1, dk, step_along(g, x, k + 1), w[0]);
      if (k < 2) plaquette(s, k, 3, dk, step_along(g, x, 3), w[0]);
      if (k == 3) plaquette(s, 0, 2, step_along(g, x, 0), step_along(g, x, 2), w[0]);
      (void)next_loop(s, w[0]);
    } else {
      // cube loops: squares 01, 01, 02, 12 carried along 2, 3, 3, 3
      const int nu = k == 3 ? 1 : 0, rho = k < 2 ? 1 : 2, mu = k == 0 ? 2 : 3;
      cube_loops(s, nu, rho, mu, step_along(g, x, nu), step_along(g, x, rho), step_along(g, x, mu), w);
      // plaquettes and rectangles: squares 01, 23 | 02, 13 | 03 | 12
      const int n1 = k == 3 ? 1 : 0, r1 = k == 0 ? 1 : k == 2 ? 3 : 2;
      square_loops(s, n1, r1, step_along(g, x, n1), step_along(g, x, r1), w);
      if (k < 2) {
        const int n2 = k == 0 ? 2 : 1;
        square_loops(s, n2, 3, step_along(g, x, n2), step_along(g, x, 3), w);
      }
    }
  }
  block_sum_store<3>(w, partials + 3 * (size_t)blockIdx.x);
}

// Deterministic two-stage reduction of the per-workgroup partials: stage 1 (kFinishGroups
// blocks) sums contiguous groups of partials, stage 2 (one block) sums the group sums,
// both in a fixed order. One block summing all 65,536 partials of the 32^3 x 64 force
// took 25 us, alone on the GPU; the two stages take about a third of that.
constexpr int kFinishGroups = 64;

__global__ __launch_bounds__(256) void finish_stage1(const double* __restrict__ act, int nact,
                                                     const double* __restrict__ kin, int nkin,
                                                     double* __restrict__ stage) {
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  const int ga = (nact + kFinishGroups - 1) / kFinishGroups, gk = (nkin + kFinishGroups - 1) / kFinishGroups;
  const int a0 = blockIdx.x * ga, a1 = min(nact, a0 + ga);
  const int k0 = blockIdx.x * gk, k1 = min(nkin, k0 + gk);
  for (int i = a0 + (int)threadIdx.x; i < a1; i += blockDim.x) {
    v[0] += act[3 * (size_t)i + 0];
    v[1] += act[3 * (size_t)i + 1];
    v[2] += act[3 * (size_t)i + 2];
  }
  for (int i = k0 + (int)threadIdx.x; i < k1; i += blockDim.x) v[3] += kin[i];
  block_sum_store<4>(v, stage + 4 * (size_t)blockIdx.x);
}

// S and W from the summed partials v: with deficit sums w_X = sum over class-X loops of
// (3 - Re tr P),
//   S = beta/3 (c_P w_P + c_R w_R + c_C w_C),  W_X = 3 n_X V - w_X  (n = 6, 12, 16).
// mode 0 writes out[0..3] = S, W_P, W_R, W_C; mode 1 adds the kinetic partials and
// writes out[0] = S + K.
__device__ __forceinline__ void finish_values(const double (&v)[4], int kind, const Coeffs& c, double V, int mode,
                                              double* __restrict__ out) {
  double wP, wR, wC, cwC;
  if (kind == 0) {  // direct force: each loop seen from 4 / 6 / 6 links
    wP = v[0] / 4.0;
    wR = v[1] / 6.0;
    wC = v[2] / 6.0;
    cwC = c.c[2] * wC;
  } else if (kind == 1) {  // action kernel: per-loop sums
    wP = v[0];
    wR = v[1];
    wC = v[2];
    cwC = c.c[2] * wC;
  } else {  // factored force: long sides see a rectangle 4 times, the mixed sum holds
            // c_R x (2 views of every rectangle) + c_C x (6 views of every cube loop);
            // W_C needs c_C != 0 (the library runs the action kernel otherwise)
    wP = v[0] / 4.0;
    wR = v[1] / 4.0;
    cwC = (v[2] - 0.5 * c.c[1] * v[1]) / 6.0;
    wC = c.c[2] != 0.0 ? cwC / c.c[2] : __builtin_nan("");
  }
  const double S = c.beta / 3.0 * (c.c[0] * wP + c.c[1] * wR + cwC);
  if (mode == 0) {
    out[0] = S;
    out[1] = 18.0 * V - wP;
    out[2] = 36.0 * V - wR;
    out[3] = 48.0 * V - wC;
  } else {
    out[0] = S + v[3];
  }
}

// Stage 2 (one block).
__global__ __launch_bounds__(64) void finish_stage2(const double* __restrict__ stage, int kind, Coeffs c, double V,
                                                    int mode, double* __restrict__ out) {
  double v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = stage[4 * (size_t)threadIdx.x + k];
  block_sum<4>(v);
  if (threadIdx.x == 0) finish_values(v, kind, c, V, mode, out);
}

// Both stages in one block, for the partials of small lattices (at most kFinishSmall: four
// per thread): one launch less, 4 us of a 4^4 force's 28.
constexpr int kFinishSmall = 1024;

__global__ __launch_bounds__(256) void finish_small(const double* __restrict__ act, int nact,
                                                    const double* __restrict__ kin, int nkin, int kind, Coeffs c,
                                                    double V, int mode, double* __restrict__ out) {
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (int i = threadIdx.x; i < nact; i += blockDim.x) {
    v[0] += act[3 * (size_t)i + 0];
    v[1] += act[3 * (size_t)i + 1];
    v[2] += act[3 * (size_t)i + 2];
  }
  for (int i = threadIdx.x; i < nkin; i += blockDim.x) v[3] += kin[i];
  block_sum<4>(v);
  if (threadIdx.x == 0) finish_values(v, kind, c, V, mode, out);
}

hipError_t finish(const double* act, int nact, const double* kin, int nkin, int kind, const Coeffs& c, double V,
                  int mode, double* stage, double* out, hipStream_t s) {
  if (nact <= kFinishSmall && nkin <= kFinishSmall) {
    finish_small<<<1, 256, 0, s>>>(act, nact, kin, nkin, kind, c, V, mode, out);
    return hipGetLastError();
  }
  finish_stage1<<<kFinishGroups, 256, 0, s>>>(act, nact, kin, nkin, stage);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  finish_stage2<<<1, kFinishGroups, 0, s>>>(stage, kind, c, V, mode, out);
  return hipGetLastError();
}

}  // namespace

int action_tiles(const Geom& g) { return site_tiles(g, kActionSites); }

template <typename T>
hipError_t launch_action(const Geom& g, const T* U, double* partials, hipStream_t s) {
  const int nt = action_tiles(g);
  action_kernel<T><<<nt, kBlock, 0, s>>>(g, U, partials, nt);
  return hipGetLastError();
}

template hipError_t launch_action<float>(const Geom&, const float*, double*, hipStream_t);
template hipError_t launch_action<double>(const Geom&, const double*, double*, hipStream_t);

hipError_t launch_finish_action(const double* partials, int nparts, int kind, const Geom& g, const Coeffs& c,
                                double* stage, double* out, hipStream_t s) {
  return finish(partials, nparts, nullptr, 0, kind, c, 2.0 * g.Vh, 0, stage, out, s);
}

hipError_t launch_finish_hamiltonian(const double* act_parts, int nact, int act_kind, const double* kin_parts,
                                     int nkin, const Geom& g, const Coeffs& c, double* stage, double* out,
                                     hipStream_t s) {
  return finish(act_parts, nact, kin_parts, nkin, act_kind, c, 2.0 * g.Vh, 1, stage, out, s);
}

}  // namespace sym
