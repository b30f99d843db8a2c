// SSOR approximate domain inverse of the SAP preconditioner (Sec. 2.2, SSOR
// equations), with the paper's naming: on a domain A_DD = 1 - Lf - Ub, Lf the
// forward in-domain hops, Ub the backward ones, and
//   B = (1 - w Ub)^{-1} [ sum_{j=0}^{N} (1 - A^S)^j ] (1 - w Lf)^{-1},
//   A^S = (1/w) [ (1 - w Lf)^{-1} + (1 - w Ub)^{-1} + (w - 2) (1 - w Lf)^{-1} (1 - w Ub)^{-1} ].
// For N = 1 (the paper's setting) B r takes four triangular sweeps:
//   t = F r,  u = G t,  c = F (t + (w - 2) u),  y = G (2 t - (u + c) / w),
// with F = (1 - w Lf)^{-1}, G = (1 - w Ub)^{-1}, since A^S t = (u + c) / w;
// N = 0 is y = G F r.  Inside SAP the residual r = eta - A psi of the domain
// is formed in the first sweep, site by site, instead of by a separate pass.
//
// A triangular solve x = in + w Lf x is a wavefront: a forward hop raises the
// hyperplane index h = l_0 + l_1 + l_2 + l_3 of the local coordinates by one,
// so all sites of a hyperplane are independent once the hyperplane above is
// done, top down for F, bottom up for G, with a barrier between hyperplanes.
//
// FP64 and FP32 storage (k_ssor_planes): one workgroup owns a domain and a few
// columns.  What a hyperplane reads of the one before it passes through LDS;
// every other field, and the links, lie in wavefront order, so that neighbouring
// lanes read neighbouring elements and the next hyperplane's links can be
// fetched ahead.  The chain of 4 (sum_mu (b_mu - 1) + 1) hyperplanes, each four
// hops and a barrier, bounds it: two neighbouring lanes share an item, each
// with one of the two spins of a hop, and trade a result where the lower spins
// need it, in the order in which one thread would add.
// FP16 storage, and domains whose hyperplanes exceed the LDS (k_ssor): one
// workgroup owns one domain and all columns; the fields stay in global memory
// (the domain's working set stays in the caches), items are (site of the
// hyperplane, column) pairs spread over the workgroup.
#include "domsolve.h"
#include "planes.h"

namespace mbbs {

template <int PR> constexpr int ssor_threads() { return PR == P64 ? 512 : 768; }

// The fields one launch touches (SAP storage precision PR, psi in PPSI).
template <int PR, int PPSI>
struct SsorFields {
  typename Store<PR>::Elem *eta, *r, *a, *b;
  float *eta_s, *r_s, *a_s, *b_s;
  typename Store<PPSI>::Elem* psi;
};

// One sweep.  MODE: input, destination, and what else happens
//   0: in = r                        -> a               (t = F r; blocked B)
//   5: in = eta - A psi at the site  -> a               (t = F r, r the SAP residual,
//                                                        computed on the fly: rmode 0 eta,
//                                                        1 outside hops only, 2 all)
//   1: in = a                        -> b               (u = G t)
//   6: in = a + (w - 2) b            -> r, and a <- 2a - (b + c)/w   (c, then s in place of t)
//   7: in = a                        -> b, psi (+)= y   (y = G s, N = 1)
//   4: in = a                        -> b, psi (+)= y   (y = G t, N = 0)
// The destination of a sweep is also what its hops read (the neighbours'
// results, one hyperplane earlier in the sweep).  In-place writes (a in
// mode 6, b in mode 7) touch only the item's own site, which no other item
// of the sweep reads.
template <int PR, int PPSI, int PL, bool FWD, int MODE>
__device__ __forceinline__ void ssor_sweep(const GeomK& k, int L, int base_site, double kappa, double omega,
                                           const SsorFields<PR, PPSI>& f, int rmode, bool assign,
                                           const LinkElem<PL>* __restrict__ U,
                                           const int* __restrict__ hp_loc, const int* __restrict__ hp_off, int nh) {
  using R = typename Store<PR>::Real;
  using RP = typename Store<PPSI>::Real;
  typename Store<PR>::Elem* X = MODE == 0 || MODE == 5 ? f.a : MODE == 6 ? f.r : f.b;
  float* X_s = MODE == 0 || MODE == 5 ? f.a_s : MODE == 6 ? f.r_s : f.b_s;
  const R wkr = (R)(omega * kappa), om = (R)omega, kap = (R)kappa;
  for (int step = 0; step < nh; ++step) {
    const int h = FWD ? nh - 1 - step : step;
    const int o0 = hp_off[h], nsite = hp_off[h + 1] - o0;
    for (int i = threadIdx.x; i < nsite * L; i += blockDim.x) {
      const int j = i / L, col = i - j * L;
      const int s = base_site + hp_loc[o0 + j];
      const SiteCtx c = site_ctx<DM>(k, s);
      const size_t base = (size_t)s * 12 * L + col, sidx = (size_t)s * L + col;
      cplx<R> acc[4][3][1];
      cplx<R> in[4][3];
      if constexpr (MODE == 5) {
        // the SAP residual eta - (psi - kappa (1+T)^-1 H psi) at this site
        load_spinor<PR, R>(f.eta, f.eta_s, base, L, sidx, in);
        if (rmode != 0) {
#pragma unroll
          for (int sp = 0; sp < 4; ++sp)
#pragma unroll
            for (int q = 0; q < 3; ++q) acc[sp][q][0] = cmake<R>(0, 0);
          if (rmode == 1) hop_sum<PPSI, PL, 1, DM, OUTSIDE, R>(k, c, f.psi, nullptr, U, L, col, acc);
          else hop_sum<PPSI, PL, 1, DM, ALL, R>(k, c, f.psi, nullptr, U, L, col, acc);
          if (k.clov) clover_apply<DM, 1, R>(k, s, acc);
          cplx<R> p[4][3];
          if (rmode == 2) {
            load_spinor<PPSI, R>(f.psi, nullptr, base, L, sidx, p);
          } else {
#pragma unroll
            for (int sp = 0; sp < 4; ++sp)
#pragma unroll
              for (int q = 0; q < 3; ++q) p[sp][q] = cmake<R>(0, 0);
          }
#pragma unroll
          for (int sp = 0; sp < 4; ++sp)
#pragma unroll
            for (int q = 0; q < 3; ++q) in[sp][q] = in[sp][q] - p[sp][q] + kap * acc[sp][q][0];
        }
      }
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int q = 0; q < 3; ++q) acc[sp][q][0] = cmake<R>(0, 0);
      // FP32 / FP16 storage: two directions' loads in flight; FP64 would spill
      if constexpr (PR == P64) hop_sum<PR, PL, 1, DM, FWD ? FWD_IN : BWD_IN, R>(k, c, X, X_s, U, L, col, acc);
      else hop_sense_sum<PR, PL, 1, DM, FWD ? FWD_IN : BWD_IN, R>(k, c, X, X_s, U, L, col, acc);
      if (k.clov) clover_apply<DM, 1, R>(k, s, acc);
      cplx<R> t[4][3], u[4][3];
      if constexpr (MODE == 0) {
        load_spinor<PR, R>(f.r, f.r_s, base, L, sidx, in);
      } else if constexpr (MODE == 1 || MODE == 4 || MODE == 7) {
        load_spinor<PR, R>(f.a, f.a_s, base, L, sidx, in);
      } else if constexpr (MODE == 6) {
        load_spinor<PR, R>(f.a, f.a_s, base, L, sidx, t);
        load_spinor<PR, R>(f.b, f.b_s, base, L, sidx, u);
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
          for (int q = 0; q < 3; ++q) in[sp][q] = t[sp][q] + (om - (R)2) * u[sp][q];
      }
      cplx<R> v[4][3];
#pragma unroll
      for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int q = 0; q < 3; ++q) v[sp][q] = in[sp][q] + wkr * acc[sp][q][0];
      store_spinor<PR, R>(X, X_s, base, L, sidx, v);
      if constexpr (MODE == 6) {
        // s = 2 t - (u + c) / w, with c as stored (what the hops of this sweep read)
        if constexpr (Store<PR>::scaled) load_spinor<PR, R>(X, X_s, base, L, sidx, v);
        const R inv = (R)1 / om;
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
          for (int q = 0; q < 3; ++q) t[sp][q] = (R)2 * t[sp][q] - inv * (u[sp][q] + v[sp][q]);
        store_spinor<PR, R>(f.a, f.a_s, base, L, sidx, t);
      }
      if constexpr (MODE == 4 || MODE == 7) {
        // psi gets the value as stored (FP16 storage: rounded), as the hops see it
        if constexpr (Store<PR>::scaled) load_spinor<PR, R>(X, X_s, base, L, sidx, v);
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const size_t e = base + (size_t)(3 * sp + q) * L;
            if (assign) {
              Store<PPSI>::st(f.psi, e, cplx<RP>{(RP)v[sp][q].re, (RP)v[sp][q].im});
            } else {
              auto pv = Store<PPSI>::ld(f.psi, e);
              Store<PPSI>::st(f.psi, e, cplx<RP>{(RP)(pv.re + (RP)v[sp][q].re), (RP)(pv.im + (RP)v[sp][q].im)});
            }
          }
      }
    }
    __syncthreads();
  }
}

// One workgroup per domain of the colour starting at s0 (domain-major order).
// rmode < 0: r holds the input; 0, 1, 2: the input is the SAP residual,
// formed in the first sweep (modes as in the SAP residual kernel).  The
// fields are written and read by other threads of the workgroup between
// barriers: no restrict / const qualifiers on them.
template <int PR, int PPSI, int PL, int LT = 0>
__global__ void __launch_bounds__(ssor_threads<PR>()) k_ssor(GeomK k, double kappa, int L, int s0, double omega,
                                                             int nssor, int assign, int rmode,
                                                             SsorFields<PR, PPSI> f,
                                                             const LinkElem<PL>* __restrict__ U,
                                                             const int* __restrict__ hp_loc,
                                                             const int* __restrict__ hp_off, int nh,
                                                             const int* __restrict__ frozen) {
  // one workgroup per domain, hence one system: block-uniform test and kappa
  const int sys = sys_of_domain(k, blockIdx.x);
  if (sys_frozen(k, frozen, sys)) return;
  if (k.kap) kappa = k.kap[sys];
  if constexpr (LT > 0) L = LT;   // compile-time element offsets for the common block width
  const int base_site = s0 + blockIdx.x * k.g.Vb;
  if (rmode < 0)
    ssor_sweep<PR, PPSI, PL, true, 0>(k, L, base_site, kappa, omega, f, rmode, assign, U, hp_loc, hp_off, nh);
  else
    ssor_sweep<PR, PPSI, PL, true, 5>(k, L, base_site, kappa, omega, f, rmode, assign, U, hp_loc, hp_off, nh);
  if (nssor == 0) {
    ssor_sweep<PR, PPSI, PL, false, 4>(k, L, base_site, kappa, omega, f, rmode, assign, U, hp_loc, hp_off, nh);
    return;
  }
  ssor_sweep<PR, PPSI, PL, false, 1>(k, L, base_site, kappa, omega, f, rmode, assign, U, hp_loc, hp_off, nh);
  ssor_sweep<PR, PPSI, PL, true, 6>(k, L, base_site, kappa, omega, f, rmode, assign, U, hp_loc, hp_off, nh);
  ssor_sweep<PR, PPSI, PL, false, 7>(k, L, base_site, kappa, omega, f, rmode, assign, U, hp_loc, hp_off, nh);
}

template <int PR, int PPSI, int PL>
static int ssor_launch(const mbbs_lattice_s* lat, const SapBuffers& b, int colour, bool assign, int rmode,
                       const int* frozen, hipStream_t st) {
  using ER = typename Store<PR>::Elem;
  using EP = typename Store<PPSI>::Elem;
  using EL = LinkElem<PL>;
  const Geom& g = lat->g;
  const EL* U = PL == P64 ? (const EL*)lat->U64dm : PL == P32 ? (const EL*)lat->U32dm : (const EL*)lat->U16dm;
  const int want = ((lat->hp_max * b.L + 63) / 64) * 64;
  const int T = std::max(64, std::min(ssor_threads<PR>(), want));
  SsorFields<PR, PPSI> f;
  f.eta = (ER*)b.eta; f.eta_s = b.eta_s;
  f.r = (ER*)b.r; f.r_s = b.r_s;
  f.a = (ER*)b.w; f.a_s = b.w_s;
  f.b = (ER*)b.x2; f.b_s = b.x2_s;
  f.psi = (EP*)b.psi;
  if (b.L == 12)
    hipLaunchKernelGGL((k_ssor<PR, PPSI, PL, 12>), dim3(g.ndom / 2), dim3(T), 0, st, lat->gk, lat->kappa, b.L,
                       colour * g.Vh, b.ssor_omega, b.nssor, (int)assign, rmode, f, U, (const int*)lat->hp_loc,
                       (const int*)lat->hp_off, lat->nh, frozen);
  else
    hipLaunchKernelGGL((k_ssor<PR, PPSI, PL>), dim3(g.ndom / 2), dim3(T), 0, st, lat->gk, lat->kappa, b.L,
                       colour * g.Vh, b.ssor_omega, b.nssor, (int)assign, rmode, f, U, (const int*)lat->hp_loc,
                       (const int*)lat->hp_off, lat->nh, frozen);
  MBBS_HIP(hipGetLastError());
  return MBBS_OK;
}

int ssor_colour(const mbbs_lattice_s* lat, const SapBuffers& b, int colour, bool assign, int rmode,
                const int* frozen, hipStream_t st) {
  MBBS_CHECK(b.ssor && b.x2 != nullptr, "SAP buffers bound without the SSOR field");
  MBBS_CHECK(b.nssor == 0 || b.nssor == 1, "N_SSOR must be 0 or 1");
  switch (b.prec) {
    case P64: return ssor_launch<P64, P64, P64>(lat, b, colour, assign, rmode, frozen, st);
    case P32: return ssor_launch<P32, P32, P32>(lat, b, colour, assign, rmode, frozen, st);
    default: return ssor_launch<P16, P32, P16>(lat, b, colour, assign, rmode, frozen, st);
  }
}

// ------------------------------------------------------ wavefronts through LDS
struct SsorPlan {
  int lg;     // columns per workgroup (divides L)
  int ncg;    // L / lg
  int spb;    // sites per pass over a hyperplane
  int thr;    // threads: 2 spb lg in whole waves
  size_t lds; // two hyperplanes
};
// FP64, and the clover term (CL), need more than the 128 registers that 1024
// threads leave each.
constexpr int ssor_plane_threads(int prec, bool CL) { return prec == P64 || CL ? 512 : 1024; }
using I0 = std::integral_constant<int, 0>;
using I1 = std::integral_constant<int, 1>;
using I2 = std::integral_constant<int, 2>;
using I3 = std::integral_constant<int, 3>;

struct SsorArgs {
  GeomK k;
  double kappa, omega;
  const int* frozen;
  void *eta, *r, *a, *b, *psi;
  const void* U;
  const uint2* nb;
  const uint4* wrap;
  const int *loc, *off;
  int lg, ncg, spb, nh, st, colour, nssor, assign, rmode;
};

// The place of the neighbour in direction MU (0xffff: none).
template <int MU> __device__ __forceinline__ unsigned ssor_nb(uint2 n) {
  return ((MU < 2 ? n.x : n.y) >> (16 * (MU & 1))) & 0xffffu;
}

// Of the lane pair that shares an item: the value by half, the other's value.
template <int U0, int U1, typename R>
__device__ __forceinline__ cplx<R> half_unit(int half, cplx<R> z) {
  if constexpr (U0 == U1) return unit_mul<U0>(z);
  const cplx<R> a = unit_mul<U0>(z), b = unit_mul<U1>(z);
  return cmake<R>(half ? b.re : a.re, half ? b.im : a.im);
}
__device__ __forceinline__ float pair_swap(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xf, 0xf, false));
}
__device__ __forceinline__ double pair_swap(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0xB1, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0xB1, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// One hop of a sweep, the half with spin `half` of the two that the link
// multiplies: its neighbour from LDS cell `cell` (component stride st), its
// link from lk; adds to spins half (up) and half + 2 (lo).
template <int PR, int MU, int FWD, typename R>
__device__ __forceinline__ void ssor_hop(const cplx<R>* sh, int st, int cell, int half,
                                         const typename RawT<PR>::T (&lk)[9 * RawT<PR>::per],
                                         cplx<R> (&up)[3], cplx<R> (&lo)[3], R& token) {
  constexpr SpinRule sr = spin_rule(MU, FWD);
  static_assert(sr.Q0 != sr.Q1, "each lower spin takes one of the two results");
  int c0 = cell + 3 * half * st, c1 = cell + 3 * (half ? sr.P1 : sr.P0) * st;
  asm volatile("" : "+v"(c0), "+v"(c1) : "v"(token));
  cplx<R> h[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) h[a] = sh[c0 + a * st] + half_unit<sr.A0, sr.A1>(half, sh[c1 + a * st]);
  cplx<R> u[3][3];
#pragma unroll
  for (int e = 0; e < 9; ++e) u[e / 3][e % 3] = raw_join<PR, R>(&lk[e * RawT<PR>::per]);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    cplx<R> x = cmake<R>(0, 0);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if constexpr (FWD) x = cmac(x, u[a][b], h[b]);
      else x = cmac_conj(x, u[b][a], h[b]);
    }
    up[a] = up[a] + x;
    if constexpr (sr.Q0 != 0) x = cmake<R>(pair_swap(x.re), pair_swap(x.im));
    lo[a] = lo[a] + half_unit<sr.B0, sr.B1>(half, x);
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) asm volatile("" : "+v"(up[a].re), "+v"(up[a].im), "+v"(lo[a].re), "+v"(lo[a].im));
  token = up[0].re;
}

// One sweep of a workgroup's domain and columns.  MODE as in ssor_sweep: 0: in ->
// a; 1: a -> b; 6: a, b -> a; 4, 7: a -> psi.  Fields: component e of cell
// (place lg + column) at e cells + cell.  Every item is handled by the same
// lanes in all sweeps, so only the hops' values cross threads, through LDS.
template <int PR, bool CL, bool FWD, int MODE, typename R = typename Store<PR>::Real>
__device__ __forceinline__ void ssor_plane_sweep(const SsorArgs& A, cplx<R>* sh, int dom, R wkr, const cplx<R>* in_f,
                                                 cplx<R>* fa, cplx<R>* fb, cplx<R>* psi) {
  constexpr int F = FWD ? 1 : 0;
  const int tid = threadIdx.x, lg = A.lg, st = A.st, Vb = A.k.g.Vb;
  const int half = tid & 1, y = (tid >> 1) / lg, c = (tid >> 1) - y * lg, cells = Vb * lg, zero = st - 1;
  const R om = (R)A.omega;
  const u4* U = (const u4*)A.U;
  const unsigned links = (unsigned)dom * (4 * link_vecs<PR>() * Vb);
  const uint2* nbt = A.nb + (FWD ? 0 : Vb);
  // a pass: sites [o0 + ch, o0 + ch + spb) of hyperplane h; passes are walked
  // hyperplane by hyperplane
  struct Pass { int h, o0, o1, ch; };
  auto open = [&](int h) { return Pass{h, A.off[h], A.off[h + 1], 0}; };
  auto next = [&](Pass p) {
    p.ch += A.spb;
    if (p.o0 + p.ch < p.o1) return p;
    const int h = FWD ? p.h - 1 : p.h + 1;
    return h < 0 || h >= A.nh ? Pass{-1, p.o0, p.o1, 0} : open(h);
  };
  // this thread's place in a pass (idle threads: the hyperplane's first)
  auto place = [&](const Pass& p) {
    const int q = p.o0 + p.ch + y;
    return y < A.spb && q < p.o1 ? q : p.o0;
  };
  R token = 0;
  // fetch the link that hop MU of the item at place p with neighbours m uses,
  // not before the hop that set the token is done
  auto fetch = [&](auto mu, int p, uint2 m, auto& l) {
    constexpr int MU = decltype(mu)::value;
    const unsigned n = ssor_nb<MU>(m);
    unsigned at = links + (unsigned)(FWD || n == 0xffffu ? p : (int)n);
    asm volatile("" : "+v"(at) : "v"(token));
    plane_link<PR, MU>(U, at, Vb, l);
  };
  Pass cur = open(FWD ? A.nh - 1 : 0), nxt = next(cur);
  int q = place(cur), qn = place(nxt);
  uint2 n = nbt[q], nn = nbt[qn];
  typename RawT<PR>::T l0[9 * RawT<PR>::per], l1[9 * RawT<PR>::per];
  fetch(I0{}, q, n, l0);
  fetch(I1{}, q, n, l1);
  int oprev = 0;   // first place of the hyperplane that the hops read
  while (cur.h >= 0) {
    const bool act = y < A.spb && cur.o0 + cur.ch + y < cur.o1;
    const Pass nx2 = nxt.h >= 0 ? next(nxt) : nxt;
    const int qn2 = place(nx2);
    const uint2 nn2 = nbt[qn2];
    // component r of this lane: row of spin half (r < 3) or half + 2
    const size_t own = (size_t)(3 * half) * cells + (q * lg + c);
    auto row = [&](int r) -> size_t { return own + (size_t)(r < 3 ? r : r + 3) * cells; };
    cplx<R> in[6], u[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) in[r] = in_f[row(r)];
    if constexpr (MODE == 6) {
#pragma unroll
      for (int r = 0; r < 6; ++r) u[r] = fb[row(r)];
    }
    if constexpr (MODE == 4 || MODE == 7) {
      if (!A.assign) {
#pragma unroll
        for (int r = 0; r < 6; ++r) u[r] = psi[row(r)];
      }
    }
    const cplx<R>* shr = sh + (((FWD ? cur.h + 1 : cur.h - 1) & 1) ? 12 * st : 0);
    cplx<R>* shw = sh + ((cur.h & 1) ? 12 * st : 0);
    cplx<R> up[3], lo[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) up[a] = lo[a] = cmake<R>(0, 0);
    auto at = [&](unsigned m) -> int { return m == 0xffffu ? zero : ((int)m - oprev) * lg + c; };
    ssor_hop<PR, 0, F, R>(shr, st, at(ssor_nb<0>(n)), half, l0, up, lo, token);
    fetch(I2{}, q, n, l0);
    ssor_hop<PR, 1, F, R>(shr, st, at(ssor_nb<1>(n)), half, l1, up, lo, token);
    fetch(I3{}, q, n, l1);
    ssor_hop<PR, 2, F, R>(shr, st, at(ssor_nb<2>(n)), half, l0, up, lo, token);
    fetch(I0{}, qn, nn, l0);
    ssor_hop<PR, 3, F, R>(shr, st, at(ssor_nb<3>(n)), half, l1, up, lo, token);
    fetch(I1{}, qn, nn, l1);
    if constexpr (CL) {
      cplx<R> acc[4][3][1];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const cplx<R> ou = cmake<R>(pair_swap(up[a].re), pair_swap(up[a].im));
        const cplx<R> ol = cmake<R>(pair_swap(lo[a].re), pair_swap(lo[a].im));
        acc[0][a][0] = half ? ou : up[a];
        acc[1][a][0] = half ? up[a] : ou;
        acc[2][a][0] = half ? ol : lo[a];
        acc[3][a][0] = half ? lo[a] : ol;
      }
      clover_apply<DM, 1, R>(A.k, dom * Vb + A.loc[q], acc);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        up[a] = half ? acc[1][a][0] : acc[0][a][0];
        lo[a] = half ? acc[3][a][0] : acc[2][a][0];
      }
    }
    const int cell = 3 * half * st + (q - cur.o0) * lg + c;
    const R inv = (R)1 / om;
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      const cplx<R> t = in[r];
      const cplx<R> x = MODE == 6 ? t + (om - (R)2) * u[r] : t;
      const cplx<R> v = x + wkr * (r < 3 ? up[r] : lo[r - 3]);
      if (act) {
        shw[cell + (r < 3 ? r : r + 3) * st] = v;
        if constexpr (MODE == 0) fa[row(r)] = v;
        else if constexpr (MODE == 1) fb[row(r)] = v;
        else if constexpr (MODE == 6) fa[row(r)] = (R)2 * t - inv * (u[r] + v);   // s = 2 t - (u + c) / w
        else psi[row(r)] = A.assign ? v : u[r] + v;
      }
    }
    if (nxt.h != cur.h) {
      oprev = cur.o0;
      lds_barrier();
    }
    cur = nxt; nxt = nx2;
    q = qn; qn = qn2;
    n = nn; nn = nn2;
  }
}

// One workgroup per (domain of the colour, group of lg columns).  rmode as in
// k_ssor.
template <int PR, bool CL>
__global__ void __launch_bounds__(ssor_plane_threads(PR, CL)) k_ssor_planes(SsorArgs A) {
  using R = typename Store<PR>::Real;
  using CV = cplx<R>;
  extern __shared__ double2 ssor_lds[];
  CV* sh = (CV*)ssor_lds;
  const GeomK& k = A.k;
  const int unit = xcd_block(blockIdx.x, gridDim.x);
  const int d = unit / A.ncg, cg = unit - d * A.ncg;
  const int sys = sys_of_domain(k, d);
  if (sys_frozen(k, A.frozen, sys)) return;
  const R kap = (R)(k.kap ? k.kap[sys] : A.kappa);
  const R wkr = (R)(A.omega * (k.kap ? k.kap[sys] : A.kappa));
  const int tid = threadIdx.x, lg = A.lg, Vb = k.g.Vb, cells = Vb * lg;
  const int dom = A.colour * (k.g.ndom / 2) + d;
  const size_t base = ((size_t)dom * A.ncg + cg) * 12 * cells;
  CV *eta = (CV*)A.eta + base, *r = (CV*)A.r + base, *a = (CV*)A.a + base, *b = (CV*)A.b + base, *psi = (CV*)A.psi + base;
  for (int i = tid; i < 24; i += blockDim.x) sh[i * A.st + A.st - 1] = cmake<R>(0, 0);
  if (A.rmode > 0) {
    // the SAP residual eta - (psi - kappa (1 + T)^-1 H psi) into r
    __shared__ int nbdom[8];   // the neighbouring domains
    if (tid < 8) {
      const int m = tid >> 1, f = tid & 1;
      const SiteCtx cf = site_ctx<DM>(k, dom * Vb + (f ? (k.g.b[m] - 1) * k.lstride[m] : 0));
      nbdom[tid] = neighbour<DM>(k, cf, m, f ? 1 : -1) / Vb;
    }
    __syncthreads();
    for (int i = tid; i < cells; i += blockDim.x) {
      const int p = i / lg, c = i - p * lg;
      const uint4 wr = A.wrap[p];
      const uint2 in_f = A.nb[p], in_b = A.nb[Vb + p];
      const int s = dom * Vb + A.loc[p];
      const SiteCtx cx = site_ctx<DM>(k, s);
      CV acc[4][3][1];
#pragma unroll
      for (int e = 0; e < 12; ++e) acc[e / 3][e % 3][0] = cmake<R>(0, 0);
      R token = 0;
      // hop (MU, FWD): whether it is summed; its data
      auto load = [&](auto mu, auto fwd, HopData<PR, PR, 1>& h) -> bool {
        constexpr int MU = decltype(mu)::value, FWD = decltype(fwd)::value;
        const bool leaves = ssor_nb<MU>(FWD ? in_f : in_b) == 0xffffu;
        if (A.rmode == 1 && !leaves) return false;
        const unsigned w = MU == 0 ? wr.x : MU == 1 ? wr.y : MU == 2 ? wr.z : wr.w;
        const int pn = FWD ? w & 0xffffu : w >> 16, dn = leaves ? nbdom[2 * MU + FWD] : dom;
        unsigned lv = (unsigned)(FWD ? dom : dn) * (4 * link_vecs<PR>() * Vb) + (FWD ? p : pn);
        size_t sv = ((size_t)dn * A.ncg + cg) * 12 * cells + pn * lg + c;
        asm volatile("" : "+v"(lv), "+v"(sv) : "v"(token));
        plane_link<PR, MU>((const u4*)A.U, lv, Vb, h.lk);
#pragma unroll
        for (int e = 0; e < 12; ++e) {
          const CV v = ((const CV*)A.psi)[sv + (size_t)e * cells];
          h.sp[2 * e] = v.re;
          h.sp[2 * e + 1] = v.im;
        }
        return true;
      };
      // (both hops of a direction in flight measured the same)
      auto dir = [&](auto mu) {
        constexpr int MU = decltype(mu)::value;
        {
          HopData<PR, PR, 1> h;
          if (load(mu, I1{}, h)) hop_compute<PR, PR, 1, ALL, MU, 1, R>(k, cx, h, acc);
          hop_settle(acc, token);
        }
        HopData<PR, PR, 1> h;
        if (load(mu, I0{}, h)) hop_compute<PR, PR, 1, ALL, MU, 0, R>(k, cx, h, acc);
        hop_settle(acc, token);
      };
      dir(I0{});
      dir(I1{});
      dir(I2{});
      dir(I3{});
      if constexpr (CL) clover_apply<DM, 1, R>(k, s, acc);
#pragma unroll
      for (int e = 0; e < 12; ++e) {
        const size_t o = (size_t)e * cells + i;
        const CV pv = A.rmode == 2 ? psi[o] : cmake<R>(0, 0);
        r[o] = eta[o] - pv + kap * acc[e / 3][e % 3][0];
      }
    }
  }
  __syncthreads();
  const CV* in = A.rmode == 0 ? eta : r;
  ssor_plane_sweep<PR, CL, true, 0>(A, sh, dom, wkr, in, a, b, psi);
  if (A.nssor == 0) {
    ssor_plane_sweep<PR, CL, false, 4>(A, sh, dom, wkr, a, a, b, psi);
    return;
  }
  ssor_plane_sweep<PR, CL, false, 1>(A, sh, dom, wkr, a, a, b, psi);
  ssor_plane_sweep<PR, CL, true, 6>(A, sh, dom, wkr, a, a, b, psi);
  ssor_plane_sweep<PR, CL, false, 7>(A, sh, dom, wkr, a, a, b, psi);
}

// Dynamic LDS of lg columns (two hyperplanes of 12 components, each with a cell
// that stays zero), and what a workgroup may have.
static size_t ssor_lds_bytes(const mbbs_lattice_s* lat, int prec, int lg) {
  return 24 * ((size_t)lat->hp_max * lg + 1) * (prec == P64 ? 16 : 8);
}
constexpr size_t SSOR_LDS = 160 * 1024 - 512;
// Links are addressed by 32-bit vector indices, places by 16 bits; for the
// number of domains see ssor_plan.
bool ssor_reads_links(const mbbs_lattice_s* lat, int prec) {
  const Geom& g = lat->g;
  return prec != P16 && g.Vb < 65535 && g.ndom / 2 / lat->nsys <= lat->ncu / 2 &&
         ssor_lds_bytes(lat, prec, 1) <= SSOR_LDS && (size_t)g.V * 4 * (prec == P64 ? 9 : 5) < (1ull << 32);
}

// Whether and how the sweeps run through LDS.  With fewer domains of a colour
// than CUs k_ssor leaves CUs idle; columns in workgroups of their own fill
// them.  From half as many domains as CUs k_ssor is level or ahead (it reads a
// link once for all columns).  FP32 / FP64, one cycle, L = 12, former -> this
// way in ms, on 256 CUs:
//   8^4 domains:  16  8.0 -> 1.4 / 12 -> 1.9,   64  6.9 -> 2.3 / 10.2 -> 3.3,
//                128  9.4 -> 6.8 / 15.0 -> 11.2,  256  12.7 -> 13.5 / 21.6 -> 22.3
//   6^4 domains: 128  3.0 -> 2.7 / 4.7 -> 4.0,  256  4.1 -> 4.4 / 6.5 -> 7.8
// N_SSOR = 0 (half the sweeps, the same residual and conversions) in FP64 with many
// columns is past the line already there: 5^4 domains, 128, L = 12 1.351 -> 1.360,
// L = 16 1.68 -> 1.79.
// Columns per workgroup: as many as the widest hyperplane leaves one wave per
// SIMD (256 lanes; 8^4 sites, 4^4 domains, L = 4: 0.89 -> 0.53 ms, 0.65 with 512),
// and in FP32, where two workgroups per CU remain, up to the thread limit.
// FP64 with the clover term spills too many registers (1.8 -> 2.9 ms).
static bool ssor_plan(const mbbs_lattice_s* lat, const SapBuffers& b, SsorPlan* p) {
  if (b.prec == P16 || (b.prec == P64 && lat->gk.clov) || !lat->Uhp[b.prec] || !lat->hp_nb) return false;
  if (((uintptr_t)b.eta | (uintptr_t)b.r | (uintptr_t)b.w | (uintptr_t)b.x2 | (uintptr_t)b.psi) & 15) return false;
  const int ncu = lat->ncu;
  // Both ways round alike, except where the compiler contracts the products of
  // boundary phases or of the clover term: there the rule looks at one system,
  // so that a batch runs its systems as they run alone.
  bool same = !lat->gk.clov;
  for (int m = 0; m < 4; ++m) same = same && lat->g.ph[m][1] == 0.0;
  const int ndom = lat->g.ndom / 2 / (same ? 1 : lat->nsys);
  if (ndom > (b.prec == P64 && b.nssor == 0 && b.L > 8 ? ncu / 4 : ncu / 2)) return false;
  int most = ssor_plane_threads(b.prec, lat->gk.clov), lg = 1;
  for (int c = 2; c <= b.L; ++c) {
    if (b.L % c || ssor_lds_bytes(lat, b.prec, c) > SSOR_LDS) continue;
    const int lanes = 2 * c * lat->hp_max;
    if (lanes <= 256 || (b.prec == P32 && lanes <= 1408 && ndom * (b.L / c) >= 2 * ncu)) lg = c;
  }
  p->lg = lg;
  p->ncg = b.L / lg;
  // more workgroups than CUs: two at a time on each, one works while the other waits
  if (lg == 1 && ndom * p->ncg > ncu) most = std::min(most, 512);
  p->spb = std::min(lat->hp_max, most / (2 * lg));
  p->thr = (2 * p->spb * lg + 63) / 64 * 64;
  p->lds = ssor_lds_bytes(lat, b.prec, lg);
  return true;
}
static DomPlan ssor_storage(const mbbs_lattice_s* lat, const SsorPlan& p) {
  DomPlan d{};
  d.G = 1;
  d.ts = lat->g.Vb;
  d.lg = p.lg;
  d.ncg = p.ncg;
  return d;
}
template <int PR, bool CL>
static int ssor_planes_launch(const mbbs_lattice_s* lat, const SapBuffers& b, const SsorPlan& p, int colour, bool assign,
                              int rmode, const int* frozen, hipStream_t st) {
  auto fn = k_ssor_planes<PR, CL>;
  // idempotent; the call is cheap beside the launch
  MBBS_HIP(hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds));
  SsorArgs a{};
  a.k = lat->gk;
  a.kappa = lat->kappa; a.omega = b.ssor_omega; a.frozen = frozen;
  a.eta = b.eta; a.r = b.r; a.a = b.w; a.b = b.x2; a.psi = b.psi;
  a.U = lat->Uhp[PR]; a.nb = lat->hp_nb; a.loc = lat->hp_loc; a.wrap = lat->hp_wrap; a.off = lat->hp_off;
  a.lg = p.lg; a.ncg = p.ncg; a.spb = p.spb; a.nh = lat->nh; a.st = lat->hp_max * p.lg + 1;
  a.colour = colour; a.nssor = b.nssor; a.assign = assign; a.rmode = rmode;
  hipLaunchKernelGGL(fn, dim3(lat->g.ndom / 2 * p.ncg), dim3(p.thr), p.lds, st, a);
  MBBS_HIP(hipGetLastError());
  return MBBS_OK;
}
static int ssor_planes(const mbbs_lattice_s* lat, const SapBuffers& b, const SsorPlan& p, int colour, bool assign,
                       int rmode, const int* frozen, hipStream_t st) {
  MBBS_CHECK(b.nssor == 0 || b.nssor == 1, "N_SSOR must be 0 or 1");
  auto go = [&](auto launch) { return launch(lat, b, p, colour, assign, rmode, frozen, st); };
  if (b.prec == P64) return go(ssor_planes_launch<P64, false>);
  return lat->gk.clov ? go(ssor_planes_launch<P32, true>) : go(ssor_planes_launch<P32, false>);
}

int ssor_sap_apply(const mbbs_lattice_s* lat, const SapBuffers& b, int ncy, const double2* in, const double2* gam,
                   double2* out, const int* frozen, hipStream_t st, Profiler* prof, bool* done) {
  SsorPlan p;
  *done = ssor_plan(lat, b, &p);
  if (!*done) return MBBS_OK;
  const DomPlan d = ssor_storage(lat, p);
  if (prof) prof->begin(MBBS_K_CONVERT);
  MBBS_TRY(dom_to(lat, b.prec, b.L, d, lat->hp_loc, in, gam, b.eta, nullptr, 0, frozen, st));
  if (prof) prof->end();
  for (int cy = 0; cy < ncy; ++cy)
    for (int col = 0; col < 2; ++col) {
      if (prof) prof->begin(MBBS_K_SSOR);
      MBBS_TRY(ssor_planes(lat, b, p, col, cy == 0, cy > 0 ? 2 : col, frozen, st));
      if (prof) prof->end();
    }
  if (prof) prof->begin(MBBS_K_CONVERT);
  MBBS_TRY(dom_from(lat, b.prec, b.L, d, lat->hp_loc, b.psi, out, nullptr, frozen, st));
  if (prof) prof->end();
  return MBBS_OK;
}

int ssor_blocked_apply(const mbbs_lattice_s* lat, const SapBuffers& b, const double2* in, double2* out,
                       hipStream_t st) {
  SsorPlan p;
  if (ssor_plan(lat, b, &p)) {
    const DomPlan d = ssor_storage(lat, p);
    MBBS_TRY(dom_to(lat, b.prec, b.L, d, lat->hp_loc, in, nullptr, b.r, nullptr, 0, nullptr, st));
    MBBS_TRY(ssor_planes(lat, b, p, 0, true, -1, nullptr, st));
    MBBS_TRY(ssor_planes(lat, b, p, 1, true, -1, nullptr, st));
    return dom_from(lat, b.prec, b.L, d, lat->hp_loc, b.psi, out, nullptr, nullptr, st);
  }
  // r holds the input on both colours; each colour's launch reads only its
  // own domains, and psi of each colour is assigned by its launch
  MBBS_TRY(sap_to(lat, b, in, nullptr, b.r, b.r_s, nullptr, st));
  MBBS_TRY(ssor_colour(lat, b, 0, true, -1, nullptr, st));
  MBBS_TRY(ssor_colour(lat, b, 1, true, -1, nullptr, st));
  return sap_from(lat, b, out, nullptr, st);
}

}  // namespace mbbs
