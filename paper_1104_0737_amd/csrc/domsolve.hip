// SAP domain solves kept on the chip (Sec. 2.2: residual eta - A psi of a
// colour's domains, nmr minimal-residual steps on each, psi += result).
//
// As launches of their own, the parts of an MR step stream about 27 field
// passes per domain solve through HBM.  Here a unit (domain x column group)
// keeps its residual r in LDS and A r in registers from the first hop to the
// last update: eta passes once, psi once per step.  Counted at 32^3 x 64 in FP32:
// vector instructions fill about half of a launch's cycles; with the exchange,
// past the L2s, memory moves 16.5 to 26.5 GB (3.5 to 5.6 TB/s) where 4.3 GB are
// compulsory.  The two, and the waits of a step in series, share the bound.
// Measured, SAP with 4 cycles of 4 steps, 8^4 domains, 12 columns: FP32 on
// 32^3 x 64 sites 79.7 -> 40.4 ms, FP64 on 16^3 x 32 10.4 -> 5.82 ms; 4^4
// domains, 8^4 sites, 4 columns (2 cycles): FP32 0.52 -> 0.17 ms.
//
// A domain that fits one workgroup (256 threads, one site and C columns each)
// needs nothing else.  A larger one is cut into G tiles with one workgroup
// each: they exchange the faces of r (projected to the two spins a hop uses)
// and the partial sums of <w, r> and <w, w> through memory, with loads and
// stores of device scope (sc1: past the per-XCD L2s), never with cache-wide
// fences.  Keeping a group's workgroups on one XCD measured the same (41.1 ms):
// that traffic passes its L2 anyway.
//
// The groups of G workgroups are formed from tickets in the order in which
// workgroups start, so only resident workgroups wait for each other: at most
// G - 1 workgroups of a launch can wait for members that have not started.
// Every wait is bounded.  One that gives up sets a word in the workspace: the
// later launches of the call then do nothing, and the closing conversion writes
// NaN to the whole result, which a solve reports as a breakdown.  (Marking the
// unit alone is not enough: its workgroups leave, and the unit that their first
// member had already claimed would keep what its psi held before.)
// Faces that carry their own validity (a mark that the reader puts back, no
// flag) took 6 % off small lattices and added 3 to 8 % to large ones, where the
// exchange's bandwidth counts; two workgroups of 256 threads per CU instead of
// one of 512 added 10 %.
//
// FP16 storage of r is left to the launches of their own: rounding r and w to
// halves costs this kernel more than it saves (3.96 -> 3.27 ms where FP32 gains
// 4.65 -> 2.74), and its rounding then differs from theirs.
#include <algorithm>

#include "domsolve.h"
#include "planes.h"

namespace mbbs {

namespace {

typedef unsigned u2 __attribute__((ext_vector_type(2)));

// Cells of a component row in LDS: TS of the tile and one that stays zero; 12
// rows for the tile (psi, then r), 6 for the projected neighbours outside it.
template <int TS> struct DomLds {
  static constexpr int ST = TS + 1, ZERO = TS, HROW = 12 * (TS + 1);
};

// Device memory of one launch's groups (G > 1).
struct DomSync {
  int* counters;              // this launch's [0] tickets, [1] units
  int* counters_next;         // the next launch's, cleared by this one
  u4* words;                  // [group][2][tile][lg][3]: a partial sum's halves, each with its tag
  unsigned long long* next;   // [group]: tag and unit to work on
  unsigned long long* flags;  // [group][tile]: tag of the faces published last
  char* slots;                // per group: the tiles' published faces
  size_t slot_bytes;
  int* lost;                  // set by a wait that gave up
  unsigned tag0;              // first tag of this launch
  int step_polls;
};

constexpr int SC1 = 16;   // device scope: coherent across the XCDs' L2 caches

__device__ __forceinline__ __amdgpu_buffer_rsrc_t dev_rsrc(void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, (unsigned)bytes, 0x00020000);
}
template <typename V>
__device__ __forceinline__ V ld_dev(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff = 0) {
  V v;
  if constexpr (sizeof(V) == 16) {
    const u4 x = __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, SC1);
    __builtin_memcpy(&v, &x, 16);
  } else if constexpr (sizeof(V) == 8) {
    const u2 x = __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, SC1);
    __builtin_memcpy(&v, &x, 8);
  } else {
    const unsigned x = __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, SC1);
    __builtin_memcpy(&v, &x, 4);
  }
  return v;
}
template <typename V>
__device__ __forceinline__ void st_dev(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff, V v) {
  if constexpr (sizeof(V) == 16) {
    u4 x;
    __builtin_memcpy(&x, &v, 16);
    __builtin_amdgcn_raw_buffer_store_b128(x, r, off, soff, SC1);
  } else if constexpr (sizeof(V) == 8) {
    u2 x;
    __builtin_memcpy(&x, &v, 8);
    __builtin_amdgcn_raw_buffer_store_b64(x, r, off, soff, SC1);
  } else {
    unsigned x;
    __builtin_memcpy(&x, &v, 4);
    __builtin_amdgcn_raw_buffer_store_b32(x, r, off, soff, SC1);
  }
}
__device__ __forceinline__ unsigned long long ld_word(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_word(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A value that all lanes read from one LDS word.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
// Wait (bounded) for a word of tag `tag`; false when the wait gave up.
__device__ __forceinline__ bool wait_word(const unsigned long long* p, unsigned tag, int polls, unsigned& low) {
  for (int i = 0; i < polls; ++i) {
    const unsigned long long v = ld_word(p);
    if ((unsigned)(v >> 32) == tag) {
      low = (unsigned)v;
      return true;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  return false;
}

// x of the lane N places further in the 16-lane row, added.
template <int N>
__device__ __forceinline__ double row_add(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x120 + N, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x120 + N, 0xf, 0xf, false);
  return x + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Sum over the lanes of the row whose index differs by a multiple of np (a
// power of two up to 8): every lane gets its sum.
__device__ __forceinline__ double row_sum(double x, int np) {
  x = row_add<8>(x);
  if (np < 8) x = row_add<4>(x);
  if (np < 4) x = row_add<2>(x);
  if (np < 2) x = row_add<1>(x);
  return x;
}

// The two spins of (1 -/+ gamma_MU) psi that a hop multiplies by the link.
template <int MU, int FWD, typename R, int C, typename V>
__device__ __forceinline__ void project(const V (&p)[12], V (&h)[6]) {
  constexpr SpinRule sr = spin_rule(MU, FWD);
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int q = 0; q < C; ++q) {
      const cplx<R> p0 = cmake<R>(p[a][2 * q], p[a][2 * q + 1]), p1 = cmake<R>(p[3 + a][2 * q], p[3 + a][2 * q + 1]);
      const cplx<R> x = cmake<R>(p[3 * sr.P0 + a][2 * q], p[3 * sr.P0 + a][2 * q + 1]);
      const cplx<R> y = cmake<R>(p[3 * sr.P1 + a][2 * q], p[3 * sr.P1 + a][2 * q + 1]);
      const cplx<R> h0 = p0 + unit_mul<sr.A0>(x), h1 = p1 + unit_mul<sr.A1>(y);
      h[a][2 * q] = h0.re; h[a][2 * q + 1] = h0.im;
      h[3 + a][2 * q] = h1.re; h[3 + a][2 * q + 1] = h1.im;
    }
}
template <typename R, int C, typename V>
__device__ __forceinline__ void project_rt(int m, int fwd, const V (&p)[12], V (&h)[6]) {
  switch (2 * m + fwd) {
    case 0: project<0, 0, R, C>(p, h); break;
    case 1: project<0, 1, R, C>(p, h); break;
    case 2: project<1, 0, R, C>(p, h); break;
    case 3: project<1, 1, R, C>(p, h); break;
    case 4: project<2, 0, R, C>(p, h); break;
    case 5: project<2, 1, R, C>(p, h); break;
    case 6: project<3, 0, R, C>(p, h); break;
    default: project<3, 1, R, C>(p, h); break;
  }
}

// One hop: the neighbour's components from LDS cell a (rows as in DomLds; a
// projected entry: components 0..5 in the halo rows, the others the zero
// cell; no neighbour: the zero cell) times the link in lk, whose successor
// (direction MN, vector ln) is fetched meanwhile.  Nothing is read before the
// hop that set `token` is done: left alone, the compiler reads all eight hops'
// data first and spills it.
template <int PR, int C, int TS, int MU, int FWD, int MN, typename R>
__device__ __forceinline__ void dom_hop(const void* lds, int a, const typename RawT<PR>::T (&lk)[9 * RawT<PR>::per],
                                        const u4* __restrict__ U, unsigned ln, int Vb,
                                        typename RawT<PR>::T (&next)[9 * RawT<PR>::per], cplx<R> (&acc)[4][3][C],
                                        R& token) {
  asm volatile("" : "+v"(a), "+v"(ln) : "v"(token));
  HopData<PR, PR, C> d;
  using V = typename ColVec<R, C>::T;
  using D = DomLds<TS>;
  const V* sh = (const V*)lds;
  const int b = (a >= D::HROW || a == D::ZERO) ? D::ZERO : a + 6 * D::ST;
#pragma unroll
  for (int e = 0; e < 12; ++e) {
    const V v = e < 6 ? sh[a + e * D::ST] : sh[b + (e - 6) * D::ST];
#pragma unroll
    for (int q = 0; q < C; ++q) {
      d.sp[(q * 12 + e) * 2] = v[2 * q];
      d.sp[(q * 12 + e) * 2 + 1] = v[2 * q + 1];
    }
  }
  if constexpr (MN >= 0) plane_link<PR, MN>(U, ln, Vb, next);
  // these reads stay above the arithmetic
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 9 * RawT<PR>::per; ++i) d.lk[i] = lk[i];
  const SiteCtx c{};
  const GeomK k{};   // (read by hops that may leave the lattice only)
  hop_compute<PR, PR, C, INSIDE, MU, FWD, R>(k, c, d, acc);
  hop_settle(acc, token);
}
// The four hops of directions M0 and M0 + 1.  cell(m, f): LDS cell; li,
// back(m): the links of the forward and the backward hop.
template <int PR, int C, int TS, int M0, typename R, typename FC, typename FB>
__device__ __forceinline__ void dom_hops(const void* lds, const u4* __restrict__ U, unsigned li, int Vb, FC cell, FB back,
                                         cplx<R> (&acc)[4][3][C], R& token) {
  typename RawT<PR>::T l0[9 * RawT<PR>::per], l1[9 * RawT<PR>::per];
  plane_link<PR, M0>(U, li, Vb, l0);
  dom_hop<PR, C, TS, M0, 1, M0, R>(lds, cell(M0, 1), l0, U, back(M0), Vb, l1, acc, token);
  dom_hop<PR, C, TS, M0, 0, M0 + 1, R>(lds, cell(M0, 0), l1, U, li, Vb, l0, acc, token);
  dom_hop<PR, C, TS, M0 + 1, 1, M0 + 1, R>(lds, cell(M0 + 1, 1), l0, U, back(M0 + 1), Vb, l1, acc, token);
  dom_hop<PR, C, TS, M0 + 1, 0, -1, R>(lds, cell(M0 + 1, 0), l1, U, li, Vb, l0, acc, token);
}
// All eight.
template <int PR, int C, int TS, typename R, typename FC, typename FB>
__device__ __forceinline__ void dom_hops8(const void* lds, const u4* __restrict__ U, unsigned li, int Vb, FC cell, FB back,
                                          cplx<R> (&acc)[4][3][C], R& token) {
  typename RawT<PR>::T l0[9 * RawT<PR>::per], l1[9 * RawT<PR>::per];
  plane_link<PR, 0>(U, li, Vb, l0);
  dom_hop<PR, C, TS, 0, 1, 0, R>(lds, cell(0, 1), l0, U, back(0), Vb, l1, acc, token);
  dom_hop<PR, C, TS, 0, 0, 1, R>(lds, cell(0, 0), l1, U, li, Vb, l0, acc, token);
  dom_hop<PR, C, TS, 1, 1, 1, R>(lds, cell(1, 1), l0, U, back(1), Vb, l1, acc, token);
  dom_hop<PR, C, TS, 1, 0, 2, R>(lds, cell(1, 0), l1, U, li, Vb, l0, acc, token);
  dom_hop<PR, C, TS, 2, 1, 2, R>(lds, cell(2, 1), l0, U, back(2), Vb, l1, acc, token);
  dom_hop<PR, C, TS, 2, 0, 3, R>(lds, cell(2, 0), l1, U, li, Vb, l0, acc, token);
  dom_hop<PR, C, TS, 3, 1, 3, R>(lds, cell(3, 1), l0, U, back(3), Vb, l1, acc, token);
  dom_hop<PR, C, TS, 3, 0, -1, R>(lds, cell(3, 0), l1, U, li, Vb, l0, acc, token);
}

// Everything a launch needs, as one kernel argument.  The kernel reads it
// through `A`, a pointer to the argument segment that is made opaque at each
// phase, so that a value is loaded again where it is used (a scalar load)
// instead of being kept, and spilled, over the whole kernel.
struct DomArgs {
  DomPlan P;
  DomSync sy;
  int nd[4], b[4], lstride[4], ndomc, nsys, ndt, Vb, fstride, colour, mode, nmr, clov;
  double kappa, ph[4][2];
  const double* kap;
  const void *eta, *U, *cinv64, *cinv32;
  void* psi;
  const int* frozen;
};
typedef const __attribute__((address_space(4))) DomArgs* DomArgsPtr;
#define DOM_RELOAD(A) asm volatile("" : "+s"(A))
__device__ __forceinline__ int dom_sys(DomArgsPtr A, int dom) { return A->nsys == 1 ? 0 : dom / (A->ndomc / A->nsys); }
__device__ __forceinline__ bool dom_frozen(DomArgsPtr A, int dom) {
  return A->frozen && A->frozen[dom_sys(A, dom) * A->fstride];
}
template <int C, typename R>
__device__ __forceinline__ void dom_clover(DomArgsPtr A, int s, cplx<R> (&acc)[4][3][C]) {
  GeomK k;
  k.cinv64[DM] = (const double*)A->cinv64;
  k.cinv32[DM] = (const float*)A->cinv32;
  clover_apply<DM, C, R>(k, s, acc);
}

// One launch: the units (domains of a colour x column groups).
// mode 0: psi = 0 everywhere, r = eta; 1: psi = 0 on this colour; 2: general.
// In modes 0 and 1 psi is assigned, else added to.
// Launch: G = 1: one workgroup per unit; else ngroups G workgroups.  TS: LDS
// cells per row, at least the workgroup's threads.  Two waves per SIMD: 256
// VGPRs per lane, and at TS = 512 one workgroup per CU.
template <int PR, int C, int TS>
__global__ void __launch_bounds__(TS, 2) k_dom(DomArgs) {
  DomArgsPtr A = (DomArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  DOM_RELOAD(A);
  using R = typename Store<PR>::Real;
  using V = typename ColVec<R, C>::T;
  using D = DomLds<TS>;
  constexpr int NF = 6;                    // components of a projected entry
  constexpr int NROW = TS / 16;            // 16-lane rows of the workgroup
  extern __shared__ float4 dom_lds[];
  V* sh = (V*)dom_lds;
  __shared__ double red[3 * 16 * NROW];    // [3][column][row of lanes]
  __shared__ double om_sh[2 * 16];
  __shared__ int ish[5];                   // group, member, a wait gave up, unit, one gave up in an earlier launch
  const int tid = threadIdx.x;
  const int nthr = blockDim.x;

  // ---- the group this workgroup belongs to: tickets are drawn as workgroups
  // start, so a group's members are resident or about to be
  int gid = 0, mem = 0;
  bool lost = false;   // a wait gave up
  if (A->P.G > 1) {
    if (tid == 0) {
      ish[4] = __hip_atomic_load(A->sy.lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int t = __hip_atomic_fetch_add(&A->sy.counters[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int g = t / A->P.G;
      ish[0] = g;
      ish[1] = t - g * A->P.G;
      ish[2] = 0;
      if (t == 0) {
        __hip_atomic_store(&A->sy.counters_next[0], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&A->sy.counters_next[1], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    lds_barrier();
    gid = uniform(ish[0]);
    mem = uniform(ish[1]);
    // (or in this one: the waits of this group's other members end too)
    if (uniform(ish[4])) return;
  }
  const __amdgpu_buffer_rsrc_t rs = dev_rsrc(A->sy.slots + (size_t)gid * A->sy.slot_bytes, A->sy.slot_bytes);
  unsigned long long* flags = A->sy.flags + (size_t)gid * A->P.G;
  unsigned tag = A->sy.tag0;

  // ---- this thread's site and columns
  const int site = tid / A->P.np, pair = tid - site * A->P.np;
  const bool act = tid < A->P.T;   // (the workgroup may hold more threads: whole waves, staged faces)
  // local coordinates (a byte each), and the site's place among the entries of
  // a face of direction m (16 bits each): packed, to stay in registers
  unsigned ltp = 0, posp[2] = {0, 0};
  {
    int q = site;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int r = q / A->P.t[m];
      ltp |= (unsigned)(q - r * A->P.t[m]) << (8 * m);
      q = r;
      const int hi = site / (A->P.tstr[m] * A->P.t[m]), lo = site - (site / A->P.tstr[m]) * A->P.tstr[m];
      posp[m >> 1] |= (unsigned)(((lo + hi * A->P.tstr[m]) * A->P.np + pair) & 0xffff) << (16 * (m & 1));
    }
  }
  auto pos = [&](int m) -> int { return (posp[m >> 1] >> (16 * (m & 1))) & 0xffff; };
  const unsigned face_bytes = (unsigned)A->P.H * NF * sizeof(V);   // published faces of a tile

  // next unit to work on (member 0 only): units of stopped systems are passed over
  auto claim = [&]() -> int {
    for (;;) {
      const int u = __hip_atomic_fetch_add(&A->sy.counters[1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (u >= A->P.units) return -1;
      if (!dom_frozen(A, u / A->P.ncg)) return u;
    }
  };
  // thread 0: the group's next unit into ish[3]
  auto next_unit = [&]() {
    int u;
    if (mem == 0) {
      u = claim();
      st_word(&A->sy.next[gid], ((unsigned long long)tag << 32) | (unsigned)u);
    } else {
      unsigned low = ~0u;
      if (!wait_word(&A->sy.next[gid], tag, lost ? 1 : A->sy.step_polls, low)) ish[2] = 1;
      u = (int)low;
    }
    ish[3] = u;
  };

  int unit;
  if (A->P.G == 1) {
    unit = xcd_block(blockIdx.x, gridDim.x);
    if (dom_frozen(A, unit / A->P.ncg)) return;
  } else {
    ++tag;
    if (tid == 0) next_unit();
    lds_barrier();
    unit = uniform(ish[3]);
  }

  cplx<R> acc[4][3][C];   // hop sums, then w = A r
  auto clear_acc = [&]() {
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int q = 0; q < C; ++q) acc[sp][a][q] = cmake<R>(0, 0);
  };

  while (unit >= 0) {
    DOM_RELOAD(A);
    const int dom = unit / A->P.ncg, cg = unit - dom * A->P.ncg;
    const int Dm = A->colour * A->ndomc + dom;
    const int sys = dom_sys(A, dom);
    const R kap = (R)(A->kap ? A->kap[sys] : A->kappa);
    // domain coordinates (as site_ctx<DM>) and neighbour domains' positions
    int dc[4];
    {
      const int id = 2 * dom;
      int q = id;
#pragma unroll
      for (int m = 0; m < 4; ++m) { const int r = q / A->nd[m]; dc[m] = m < 3 ? q - r * A->nd[m] : q; q = r; }
      if (((dc[0] + dc[1] + dc[2] + dc[3]) & 1) != A->colour) dc[0] += 1;
    }
    // first vectors of a domain's links
    auto links = [&](int d) -> unsigned { return (unsigned)d * (4 * link_vecs<PR>() * A->Vb); };
    auto other_dom = [&](int m, int f, bool& wrap) -> int {
      const int lo = m == 3 ? sys * A->ndt : 0, nd = m == 3 ? A->ndt : A->nd[m];
      int c[4] = {dc[0], dc[1], dc[2], dc[3]};
      const int nv = c[m] + (f ? 1 : -1);
      wrap = nv < lo || nv == lo + nd;
      c[m] = nv < lo ? lo + nd - 1 : (nv == lo + nd ? lo : nv);
      const int id = c[0] + A->nd[0] * (c[1] + A->nd[1] * (c[2] + A->nd[2] * c[3]));
      return (1 - A->colour) * A->ndomc + (id >> 1);
    };
    // this workgroup's tile of the domain
    const int tl = mem;
    int tc[4], loc = 0;
    int me = act ? tid : 0;
    unsigned code = 0;      // per hop (m, f) two bits: 0 none, 1 in the tile, 2 in another tile
    {
      int q = tl;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int r = q / A->P.nt[m];
        tc[m] = q - r * A->P.nt[m];
        q = r;
        const int l = (ltp >> (8 * m)) & 0xff;
        loc += (tc[m] * A->P.t[m] + l) * A->lstride[m];
        const int below = l > 0 ? 1 : (tc[m] > 0 ? 2 : 0);
        const int above = l < A->P.t[m] - 1 ? 1 : (tc[m] < A->P.nt[m] - 1 ? 2 : 0);
        code |= (unsigned)(below | (above << 2)) << (4 * m);
      }
      if (!act) { loc = 0; code = 0; }
    }
    unsigned li = links(Dm) + loc;
    // first element of the tile (in column vectors)
    const size_t own = ((((size_t)Dm * A->P.ncg + cg) * A->P.G + tl) * 12) * A->P.T;
    // publish the faces of r (in v) that other tiles of the domain read
    auto publish = [&](const V (&v)[12]) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        if (A->P.nt[m] == 1) continue;
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          // f = 1: the low face, read by the tile below for its forward hop
          if (((code >> (4 * m + 2 * (1 - f))) & 3) != 2) continue;
          // region of the reading hop: low faces where the reader keeps its
          // forward entries, high faces where it keeps its backward ones
          const unsigned off = tl * face_bytes + (unsigned)(A->P.hoff[m][f] * NF + pos(m)) * sizeof(V);
          const unsigned step = A->P.n[m] * sizeof(V);
          V w[6];
          if (f) { if (m == 0) project<0, 1, R, C>(v, w); else if (m == 1) project<1, 1, R, C>(v, w);
                   else if (m == 2) project<2, 1, R, C>(v, w); else project<3, 1, R, C>(v, w); }
          else   { if (m == 0) project<0, 0, R, C>(v, w); else if (m == 1) project<1, 0, R, C>(v, w);
                   else if (m == 2) project<2, 0, R, C>(v, w); else project<3, 0, R, C>(v, w); }
#pragma unroll
          for (int e = 0; e < NF; ++e) st_dev<V>(rs, off, e * step, w[e]);
        }
      }
    };
    // all of the workgroup's published faces are in memory: tell the readers
    auto published = [&](unsigned tg) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      lds_barrier();
      if (tid == 0) st_word(&flags[tl], (unsigned long long)tg << 32);
    };

    // ---- the SAP residual r = eta - psi + kappa H psi
    ++tag;
    {
      if (A->mode != 0) {
        for (int e = tid; e < 6; e += nthr) sh[e * D::ST + D::ZERO] = V(0);
        if (A->mode == 2) {
          V p[12];
#pragma unroll
          for (int e = 0; e < 12; ++e) p[e] = ((V*)A->psi + own + e * A->P.T)[me];
          if (act) {
#pragma unroll
            for (int e = 0; e < 12; ++e) sh[e * D::ST + tid] = p[e];
          }
        }
        clear_acc();
        // the faces outside the tile that directions m0 and m0 + 1 read: staged
        // in two parts, to fit the halo rows
        auto stage = [&](int m0) {
          const int n0 = A->P.n[m0], n1 = A->P.n[m0 + 1];
          if (tid < 2 * (n0 + n1)) {
            const int m = tid < 2 * n0 ? m0 : m0 + 1;
            const int rem = tid < 2 * n0 ? tid : tid - 2 * n0, nm = tid < 2 * n0 ? n0 : n1;
            const int f = rem >= nm, q = rem - f * nm;
            const int fs = q / A->P.np, pr = q - fs * A->P.np;
            const int ts_m = m == 0 ? A->P.tstr[0] : m == 1 ? A->P.tstr[1] : m == 2 ? A->P.tstr[2] : A->P.tstr[3];
            const int t_m = m == 0 ? A->P.t[0] : m == 1 ? A->P.t[1] : m == 2 ? A->P.t[2] : A->P.t[3];
            const int nt_m = m == 0 ? A->P.nt[0] : m == 1 ? A->P.nt[1] : m == 2 ? A->P.nt[2] : A->P.nt[3];
            const int tg_m = m == 0 ? A->P.tgs[0] : m == 1 ? A->P.tgs[1] : m == 2 ? A->P.tgs[2] : A->P.tgs[3];
            const int tc_m = m == 0 ? tc[0] : m == 1 ? tc[1] : m == 2 ? tc[2] : tc[3];
            const int hi = fs / ts_m, lo = fs - hi * ts_m;
            const int sn = lo + (f ? 0 : t_m - 1) * ts_m + hi * ts_m * t_m;   // the neighbour's site in its tile
            const bool in = f ? tc_m < nt_m - 1 : tc_m > 0;
            bool wrap = false;
            const int Dn = in ? Dm : other_dom(m, f, wrap);
            const int tn = in ? tl + (f ? tg_m : -tg_m) : tl + (f ? -(nt_m - 1) * tg_m : (nt_m - 1) * tg_m);
            V h[6];
#pragma unroll
            for (int e = 0; e < 6; ++e) h[e] = V(0);
            if (A->mode == 2 || !in) {
              const V* src = (const V*)A->psi + ((((size_t)Dn * A->P.ncg + cg) * A->P.G + tn) * 12) * A->P.T + (sn * A->P.np + pr);
              V p[12];
#pragma unroll
              for (int e = 0; e < 12; ++e) p[e] = src[(size_t)e * A->P.T];
              project_rt<R, C>(m, f, p, h);
              if (wrap) {
                const cplx<R> ph = cmake<R>((R)A->ph[m][0], (R)(f ? A->ph[m][1] : -A->ph[m][1]));
#pragma unroll
                for (int e = 0; e < 6; ++e)
#pragma unroll
                  for (int q2 = 0; q2 < C; ++q2) {
                    const cplx<R> x = ph * cmake<R>(h[e][2 * q2], h[e][2 * q2 + 1]);
                    h[e][2 * q2] = x.re; h[e][2 * q2 + 1] = x.im;
                  }
              }
            }
#pragma unroll
            for (int e = 0; e < 6; ++e) sh[D::HROW + e * D::ST + tid] = h[e];
          }
        };
        auto cell = [&](int m, int f) -> int {
          const unsigned c = (code >> (4 * m + 2 * f)) & 3;
          if (c == 1) return A->mode == 2 ? tid + (f ? A->P.tstr[m] : -A->P.tstr[m]) * A->P.np : D::ZERO;
          return D::HROW + ((m & 1) ? 2 * A->P.n[m - 1] : 0) + f * A->P.n[m] + pos(m);
        };
        auto back = [&](int m) -> unsigned {
          if ((code >> (4 * m)) & 3) return li - A->lstride[m];
          bool w;
          return links(other_dom(m, 0, w)) + loc + (A->b[m] - 1) * A->lstride[m];
        };
        R token = 0;
        stage(0);
        lds_barrier();
        if (act) dom_hops<PR, C, TS, 0, R>(sh, (const u4*)A->U, li, A->Vb, cell, back, acc, token);
        lds_barrier();
        stage(2);
        lds_barrier();
        if (act) {
          dom_hops<PR, C, TS, 2, R>(sh, (const u4*)A->U, li, A->Vb, cell, back, acc, token);
          if (A->clov) dom_clover<C, R>(A, Dm * A->Vb + loc, acc);
        }
      }
#pragma unroll
      for (int e = 0; e < 12; ++e) {
        const V ev = ((const V*)A->eta + own + e * A->P.T)[me];
        const V pv = A->mode == 2 ? sh[e * D::ST + me] : V(0);
#pragma unroll
        for (int q = 0; q < C; ++q) {
          cplx<R> x = cmake<R>(ev[2 * q], ev[2 * q + 1]);
          if (A->mode != 0) x = x - cmake<R>(pv[2 * q], pv[2 * q + 1]) + kap * acc[e / 3][e % 3][q];
          acc[e / 3][e % 3][q] = x;
        }
      }
    }
    // r (in acc) to LDS, its faces to the other tiles; `fresh`: LDS held psi
    auto put_r = [&](bool fresh) {
      V r[12];
#pragma unroll
      for (int e = 0; e < 12; ++e)
#pragma unroll
        for (int q = 0; q < C; ++q) { r[e][2 * q] = acc[e / 3][e % 3][q].re; r[e][2 * q + 1] = acc[e / 3][e % 3][q].im; }
      if (fresh) {
        lds_barrier();   // psi's rows are read until here
        for (int e = tid; e < 6; e += nthr) sh[e * D::ST + D::ZERO] = V(0);
      }
      if (act) {
#pragma unroll
        for (int e = 0; e < 12; ++e) sh[e * D::ST + tid] = r[e];
      }
      if (A->P.G > 1) publish(r);
    };
    put_r(true);
    if (A->P.G > 1) published(tag);
    lds_barrier();

    // ---- the MR steps
    for (int step = 0; step < A->nmr; ++step) {
      const unsigned ftag = tag;   // tag of the faces of this step's r
      // opaque per step: addresses derived from these are formed where they are
      // used instead of being kept in registers over all steps
      asm volatile("" : "+v"(posp[0]), "+v"(posp[1]), "+v"(ltp), "+v"(code), "+v"(li), "+v"(loc), "+v"(me));
      DOM_RELOAD(A);
      // two sets of words in turn: a workgroup may reach the next step's sums
      // while another still reads this step's
      const unsigned nwords = A->P.G * A->P.lg * 3;
      const __amdgpu_buffer_rsrc_t wrs =
          dev_rsrc(A->sy.words + ((size_t)gid * 2 + (tag >> 1 & 1)) * nwords, nwords * sizeof(u4));
      ++tag;
      if (A->P.G > 1) {
        // the faces of the neighbouring tiles
        if (tid < 8) {
          const int m = tid >> 1, f = tid & 1;
          const int nt_m = A->P.nt[m], tc_m = m == 0 ? tc[0] : m == 1 ? tc[1] : m == 2 ? tc[2] : tc[3];
          if (f ? tc_m < nt_m - 1 : tc_m > 0) {
            unsigned low;
            if (!wait_word(&flags[tl + (f ? A->P.tgs[m] : -A->P.tgs[m])], ftag, lost ? 1 : A->sy.step_polls, low)) ish[2] = 1;
          }
        }
        lds_barrier();
        asm volatile("" ::: "memory");
        if (tid < A->P.H) {
          // entry tid of the halo: its direction and side
          int m = -1, f = 0;
#pragma unroll
          for (int mm = 0; mm < 4; ++mm)
#pragma unroll
            for (int ff = 0; ff < 2; ++ff) {
              const bool has = ff ? tc[mm] < A->P.nt[mm] - 1 : tc[mm] > 0;
              if (has && tid >= A->P.hoff[mm][ff] && tid < A->P.hoff[mm][ff] + A->P.n[mm]) { m = mm; f = ff; }
            }
          if (m >= 0) {
            const int nm = A->P.n[m];
            const unsigned off = (unsigned)(tl + (f ? A->P.tgs[m] : -A->P.tgs[m])) * face_bytes +
                                 (unsigned)(A->P.hoff[m][f] * NF + (tid - A->P.hoff[m][f])) * sizeof(V);
            V h[NF];
#pragma unroll
            for (int e = 0; e < NF; ++e) h[e] = ld_dev<V>(rs, off + (unsigned)(e * nm) * sizeof(V));
#pragma unroll
            for (int e = 0; e < NF; ++e) sh[D::HROW + e * D::ST + tid] = h[e];
          }
        }
        lds_barrier();
      }
      auto cell = [&](int m, int f) -> int {
        const unsigned c = (code >> (4 * m + 2 * f)) & 3;
        if (c == 1) return tid + (f ? A->P.tstr[m] : -A->P.tstr[m]) * A->P.np;
        if (c == 2) return D::HROW + A->P.hoff[m][f] + pos(m);
        return D::ZERO;
      };
      auto back = [&](int m) -> unsigned { return ((code >> (4 * m)) & 3) ? li - A->lstride[m] : li; };
      double sums[C][3];
#pragma unroll
      for (int q = 0; q < C; ++q) sums[q][0] = sums[q][1] = sums[q][2] = 0;
      if (act) {
        R token = 0;
        clear_acc();
        dom_hops8<PR, C, TS, R>(dom_lds, (const u4*)A->U, li, A->Vb, cell, back, acc, token);
        if (A->clov) dom_clover<C, R>(A, Dm * A->Vb + loc, acc);
        // w = r - kappa H r, and <w, r>, <w, w>
        R a_re[C], a_im[C], a_ww[C];
#pragma unroll
        for (int q = 0; q < C; ++q) a_re[q] = a_im[q] = a_ww[q] = 0;
#pragma unroll
        for (int e = 0; e < 12; ++e) {
          const V v = sh[e * D::ST + tid];
#pragma unroll
          for (int q = 0; q < C; ++q) {
            const cplx<R> y = cmake<R>(v[2 * q], v[2 * q + 1]);
            const cplx<R> x = y - kap * acc[e / 3][e % 3][q];
            acc[e / 3][e % 3][q] = x;
            a_re[q] = fmar(x.re, y.re, fmar(x.im, y.im, a_re[q]));
            a_im[q] = fmar(x.re, y.im, fmar(-x.im, y.re, a_im[q]));
            a_ww[q] = fmar(x.re, x.re, fmar(x.im, x.im, a_ww[q]));
          }
        }
#pragma unroll
        for (int q = 0; q < C; ++q) { sums[q][0] = a_re[q]; sums[q][1] = a_im[q]; sums[q][2] = a_ww[q]; }
      }
      // sums over the tile's sites per column, in a fixed order: rows of 16
      // lanes, then the rows
#pragma unroll
      for (int q = 0; q < C; ++q)
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          const double x = row_sum(sums[q][m], A->P.np);
          if ((tid & 15) < A->P.np) red[(m * 16 + (tid & 15) * C + q) * NROW + (tid >> 4)] = x;
        }
      lds_barrier();
      const bool assign = step == 0 && A->mode != 2;
      // psi, on its way while the sums are (after them: FP64 6.05 instead of 5.98
      // ms, FP32 41.1 instead of 40.6 at the sizes above)
      V ps[12];
      if (act && !assign) {
#pragma unroll
        for (int e = 0; e < 12; ++e) ps[e] = ((V*)A->psi + own + e * A->P.T)[me];
      }
      const bool last = step + 1 == A->nmr;
      const int lg = A->P.lg, nrow = nthr >> 4;
      // thread (column, 16 lanes): total of the tile; then of the domain
      if (tid < lg * 16) {
        const int col = tid >> 4, j = tid & 15;
        double t3[3];
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          double x = 0;
          for (int y = j; y < nrow; y += 16) x += red[(m * 16 + col) * NROW + y];
          t3[m] = row_sum(x, 1);
        }
        if (A->P.G > 1) {
          if (j < 3) {
            const double x = j == 0 ? t3[0] : j == 1 ? t3[1] : t3[2];
            const unsigned long long bits = (unsigned long long)__double_as_longlong(x);
            const u4 w = {(unsigned)bits, tag, (unsigned)(bits >> 32), tag};
            st_dev<u4>(wrs, ((tl * lg + col) * 3 + j) * sizeof(u4), 0, w);
          }
          // every tile's sums: their arrival also says that the tile is done
          // with the faces
#pragma unroll
          for (int m = 0; m < 3; ++m) t3[m] = 0;
          for (int g = j; g < A->P.G; g += 16) {
            const unsigned off = (g * lg + col) * 3 * sizeof(u4);
            u4 w[3];
            bool ok;
            int polls = lost ? 1 : A->sy.step_polls;
            do {
#pragma unroll
              for (int m = 0; m < 3; ++m) w[m] = ld_dev<u4>(wrs, off + m * sizeof(u4));
              ok = w[0].y == tag && w[0].w == tag && w[1].y == tag && w[1].w == tag && w[2].y == tag && w[2].w == tag;
              asm volatile("" ::: "memory");   // read again next time
            } while (!ok && --polls > 0);
            if (!ok) ish[2] = 1;
#pragma unroll
            for (int m = 0; m < 3; ++m)
              t3[m] += __longlong_as_double((long long)(((unsigned long long)w[m].z << 32) | w[m].x));
          }
#pragma unroll
          for (int m = 0; m < 3; ++m) t3[m] = row_sum(t3[m], 1);
        }
        if (j == 0) {
          om_sh[2 * col] = t3[2] > 0 ? t3[0] / t3[2] : 0.0;
          om_sh[2 * col + 1] = t3[2] > 0 ? t3[1] / t3[2] : 0.0;
        }
      }
      if (A->P.G > 1 && last && tid == 0) next_unit();
      lds_barrier();
      if (A->P.G > 1) lost = lost || uniform(ish[2]);
      cplx<R> om[C];
#pragma unroll
      for (int q = 0; q < C; ++q) {
        const int col = (act ? pair : 0) * C + q;
        om[q] = cmake<R>((R)om_sh[2 * col], (R)om_sh[2 * col + 1]);
      }
      if (!last) ++tag;
      // psi += omega r; r -= omega w (r first: its faces travel meanwhile)
      {
        cplx<R> x[4][3][C];   // r before the update
#pragma unroll
        for (int e = 0; e < 12; ++e) {
          const V v = sh[e * D::ST + me];
#pragma unroll
          for (int q = 0; q < C; ++q) {
            x[e / 3][e % 3][q] = cmake<R>(v[2 * q], v[2 * q + 1]);
            acc[e / 3][e % 3][q] = x[e / 3][e % 3][q] - mr_mul(om[q], acc[e / 3][e % 3][q]);
          }
        }
        if (!last) put_r(false);
        if (act) {
#pragma unroll
          for (int e = 0; e < 12; ++e)
#pragma unroll
            for (int q = 0; q < C; ++q) {
              const cplx<R> d = mr_mul(om[q], x[e / 3][e % 3][q]);
              if (assign) { ps[e][2 * q] = d.re; ps[e][2 * q + 1] = d.im; }
              else { ps[e][2 * q] = ps[e][2 * q] + d.re; ps[e][2 * q + 1] = ps[e][2 * q + 1] + d.im; }
            }
          // (the result becomes NaN in any case; without this branch the compiler
          // orders the update worse: FP32 32^3 x 64 40.4 -> 41.5 ms)
          if (lost) {
#pragma unroll
            for (int e = 0; e < 12; ++e) ps[e] = V(__builtin_nanf(""));
          }
        }
        if (!last && A->P.G > 1) published(tag);
        if (act) {
#pragma unroll
          for (int e = 0; e < 12; ++e) ((V*)A->psi + own + e * A->P.T)[me] = ps[e];
        }
      }
      if (last || A->P.G == 1) lds_barrier();
    }
    if (A->P.G == 1) break;
    unit = uniform(ish[3]);
    if (lost) unit = -1;
    lds_barrier();
  }
  if (A->P.G > 1 && tid == 0 && ish[2]) __hip_atomic_store(A->sy.lost, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------- conversions
// Blocks of SB consecutive sites of the (domain, tile, site) order.
struct DomSite { int lex, sys; size_t tile; int site; };
__device__ __forceinline__ DomSite dom_site(const GeomK& k, const DomPlan& P, const int* __restrict__ order, int q) {
  DomSite d;
  const int tile_g = q / P.ts;            // tile over the lattice
  d.site = q - tile_g * P.ts;
  const int D = tile_g / P.G, tile = tile_g - D * P.G;
  int a = d.site, b = tile, loc = 0;
  if (order) {
    loc = order[d.site];
  } else {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int ra = a / P.t[m], rb = b / P.nt[m];
      loc += ((b - rb * P.nt[m]) * P.t[m] + (a - ra * P.t[m])) * k.lstride[m];
      a = ra; b = rb;
    }
  }
  const SiteCtx c = site_ctx<DM>(k, D * k.g.Vb + loc);
  d.lex = lex_of(k, c);
  d.sys = c.sys;
  // first element of (domain, column group 0, tile): the groups follow G tiles apart
  d.tile = ((size_t)D * P.ncg) * P.G + tile;
  return d;
}

// FP64 lexicographic block (times gam) -> storage of this path.  The sites'
// rows pass through LDS: read as whole rows, written as runs of sites.  The
// first block also clears the launches' counters and tags.
template <int PR, int LT = 0>
__global__ void __launch_bounds__(256) k_to_dom(GeomK k, DomPlan P, int L, int SB, const double2* __restrict__ in,
                                                const double2* __restrict__ gam, typename Store<PR>::Elem* __restrict__ out,
                                                unsigned* __restrict__ clear, int nclear,
                                                const int* __restrict__ order, const int* __restrict__ frozen) {
  if constexpr (LT > 0) L = LT;
  using R = typename Store<PR>::Real;
  extern __shared__ double2 gsh[];
  __shared__ DomSite ds[16];
  const int tid = threadIdx.x, nthr = blockDim.x;
  for (int i = blockIdx.x * nthr + tid; i < nclear; i += gridDim.x * nthr) clear[i] = 0;
  const int q0 = blockIdx.x * SB;
  if (tid < SB) ds[tid] = dom_site(k, P, order, q0 + tid);
  __syncthreads();
  // SB divides the domain volume: one system per block
  const int sys = ds[0].sys;
  if (sys_frozen(k, frozen, sys)) return;
  double2* ish = gsh + (gam ? L * L : 0);
  if (gam)
    for (int e = tid; e < L * L; e += nthr) gsh[e] = gam[(size_t)sys * L * L + e];
  const int row = 12 * L, tot_e = SB * row;
  constexpr int NB = 8;
  for (int f0 = tid; f0 < tot_e; f0 += NB * nthr) {
    double2 buf[NB];
    int ff[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      ff[j] = min(f0 + j * nthr, tot_e - 1);
      const int y = ff[j] / row, w = ff[j] - y * row;
      buf[j] = in[(size_t)ds[y].lex * row + w];
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) ish[ff[j]] = buf[j];
  }
  __syncthreads();
  if (tid >= SB * L) return;
  // thread -> (column group, site, column of the group)
  const int lg = P.lg, c = tid % lg, y = (tid / lg) % SB, cg = tid / (lg * SB), j = cg * lg + c;
  const double2* xr = ish + (size_t)y * row;
  cplx<R> v[4][3];
  if (gam && LT > 0) {
    // this thread's column of gam in registers: half the product's LDS reads
    // (32^3 x 64, L = 12, FP32: 3.80 -> 3.35 ms; 1.39 ms without gam)
    cplx<double> g[LT > 0 ? LT : 1];
#pragma unroll
    for (int m = 0; m < LT; ++m) g[m] = cmake(gsh[m * L + j].x, gsh[m * L + j].y);
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        cplx<double> acc = cmake(0.0, 0.0);
#pragma unroll
        for (int m = 0; m < LT; ++m) {
          const double2 e = xr[(3 * sp + a) * L + m];
          acc = acc + cmake(e.x, e.y) * g[m];
        }
        v[sp][a] = cmake<R>((R)acc.re, (R)acc.im);
      }
  } else if (gam) {
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        cplx<double> acc = cmake(0.0, 0.0);
        for (int m = 0; m < L; ++m) {
          const double2 e = xr[(3 * sp + a) * L + m], g = gsh[m * L + j];
          acc = acc + cmake(e.x, e.y) * cmake(g.x, g.y);
        }
        v[sp][a] = cmake<R>((R)acc.re, (R)acc.im);
      }
  } else {
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double2 e = xr[(3 * sp + a) * L + j];
        v[sp][a] = cmake<R>((R)e.x, (R)e.y);
      }
  }
  const size_t cell = (size_t)P.ts * lg;
  const size_t blk = ds[y].tile + (size_t)cg * P.G;
  store_spinor<PR, R>(out, nullptr, blk * 12 * cell + (size_t)ds[y].site * lg + c, (int)cell, 0, v);
}

template <typename R>
__global__ void __launch_bounds__(256) k_from_dom(GeomK k, DomPlan P, int L, int SB, const cplx<R>* __restrict__ in,
                                                  double2* __restrict__ out, const int* __restrict__ order,
                                                  const int* __restrict__ lost, const int* __restrict__ frozen) {
  extern __shared__ double2 gsh[];
  __shared__ DomSite ds[16];
  cplx<R>* ish = (cplx<R>*)gsh;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int q0 = blockIdx.x * SB;
  if (tid < SB) ds[tid] = dom_site(k, P, order, q0 + tid);
  __syncthreads();
  if (sys_frozen(k, frozen, ds[0].sys)) return;
  const int lg = P.lg, row = 12 * L;
  if (tid < SB * L) {
    const int c = tid % lg, y = (tid / lg) % SB, cg = tid / (lg * SB), j = cg * lg + c;
    const size_t cell = (size_t)P.ts * lg;
    const cplx<R>* p = in + (ds[y].tile + (size_t)cg * P.G) * 12 * cell + (size_t)ds[y].site * lg + c;
    cplx<R> v[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) v[e] = p[(size_t)e * cell];
#pragma unroll
    for (int e = 0; e < 12; ++e) ish[(size_t)y * row + e * L + j] = v[e];
  }
  __syncthreads();
  const bool nan = lost && *lost;
  for (int f = tid; f < SB * row; f += nthr) {
    const int y = f / row, w = f - y * row;
    out[(size_t)ds[y].lex * row + w] = nan ? make_double2(__builtin_nan(""), __builtin_nan(""))
                                           : make_double2((double)ish[f].re, (double)ish[f].im);
  }
}

int conv_sites(int Vb, int L) {
  int best = 1;
  for (int s = 1; s <= 16 && s * L <= 256; ++s)
    if (Vb % s == 0) best = s;
  return best;
}

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }
size_t vec_bytes(int prec, int C) { return prec == P64 ? 16 : 8 * (size_t)C; }
size_t lds_bytes(int prec, int C, int TS) { return (size_t)18 * (TS + 1) * vec_bytes(prec, C); }
size_t slot_bytes(const DomPlan& p, int prec) {
  return al((size_t)p.G * p.H * 6 * vec_bytes(prec, p.C));
}
// Words cleared before the first launch: two sets of counters, the word of lost
// waits, then (16-byte aligned) the tagged partial sums, next units and face
// flags of the groups.
constexpr int SYNC_LOST = 4, SYNC_WORDS = 8;
size_t sync_ints(const DomPlan& p) {
  return SYNC_WORDS + (size_t)p.ngroups * (8 * (size_t)p.G * 3 * p.lg + 2 * (1 + (size_t)p.G));
}
// Face sizes, strides and halo places of a tile shape; false where its halo
// or the residual's staged faces exceed the LDS rows.
bool shape_tile(const Geom& g, const int (&t)[4], int np, DomPlan* p) {
  p->ts = 1; p->G = 1; p->H = 0;
  for (int m = 0; m < 4; ++m) {
    p->t[m] = t[m];
    p->nt[m] = g.b[m] / t[m];
    p->tstr[m] = p->ts;
    p->tgs[m] = p->G;
    p->ts *= t[m];
    p->G *= p->nt[m];
  }
  for (int m = 0; m < 4; ++m) {
    p->n[m] = p->ts / t[m] * np;
    p->hoff[m][0] = p->hoff[m][1] = p->H;
    if (p->nt[m] >= 2) p->H += p->n[m];
    if (p->nt[m] >= 3) { p->hoff[m][1] = p->H; p->H += p->n[m]; }
  }
  p->T = p->ts * np;
  return p->T <= p->TS && p->H <= p->TS && 2 * (p->n[0] + p->n[1]) <= p->TS && 2 * (p->n[2] + p->n[3]) <= p->TS;
}

// The tile shape for np column chunks per site: the fewest workgroups (the
// least exchange), then the smallest halo.
bool pick_shape(const Geom& g, int np, int TS, DomPlan* out) {
  bool found = false;
  for (int a = 1; a <= g.b[0]; ++a)
    for (int b = 1; g.b[0] % a == 0 && b <= g.b[1] && a * b * np <= TS; ++b)
      for (int c = 1; g.b[1] % b == 0 && c <= g.b[2] && a * b * c * np <= TS; ++c)
        for (int d = 1; g.b[2] % c == 0 && d <= g.b[3] && a * b * c * d * np <= TS; ++d) {
          if (g.b[3] % d) continue;
          DomPlan p{};
          p.TS = TS;
          const int t[4] = {a, b, c, d};
          if (!shape_tile(g, t, np, &p)) continue;
          if (!found || p.G < out->G || (p.G == out->G && p.H < out->H)) { *out = p; found = true; }
        }
  return found;
}

// Whether a plan is at least as fast as the launches it stands for.  A slot of
// TS cells takes a step's time however few of its lanes work, so the fraction
// of busy lanes decides; a group pays for its exchanges, which few steps do not
// earn back; domains of a few sites have little but launches to save.  Former
// launches' time / this form's, over 93 shapes (4096 to 10^6 sites, 1 to 13 000
// sites a domain), 1 to 32 columns, both precisions, 1 to 4 cycles:
//   one workgroup, at least half its lanes busy, or 0.3 and 32 sites: 2 steps
//   and more 1.07 to 7.0, 1 step 0.86 to 3.3 (all lanes busy 0.98 to 3.3);
//   2 to 4 workgroups as busy: 3 steps and more 1.01 to 10.6, 2 steps 0.94 to
//   6.8 (all lanes 1.06 to 6.1), 1 step 0.72 to 4.7;
//   more workgroups, 0.6 busy: 3 steps and more 1.13 to 13, 2 steps with all
//   lanes 1.21 to 3.3, 1 step 0.69 to 6.2; 0.56 busy 0.93;
//   the others at 4 steps: one workgroup 0.08 to 3.3 (1^4 domains 0.08, 2^4
//   0.25), 2 to 4 0.68 to 4.6, more 0.10 to 4.7 (5^4 0.57).
// (The gains among those lie where one round of workgroups holds all units; a
// rule with rounds would run a batch's systems in another form than each alone.)
bool dom_pays(const DomPlan& p, int Vb, int nmr) {
  const bool all = p.T == p.TS, busy = 2 * p.T >= p.TS || (10 * p.T >= 3 * p.TS && Vb >= 32);
  if (p.G == 1) return nmr == 1 ? all : busy;
  if (nmr <= 2) return nmr == 2 && all;
  return p.G <= 4 ? busy : 10 * p.T >= 6 * p.TS;
}

template <int PR, int C, int TS>
int launch_dom_ts(const mbbs_lattice_s* lat, const SapBuffers& b, const DomPlan& p, int colour, int mode, int nmr,
                  const DomSync& sy, const int* frozen, hipStream_t st) {
  auto fn = k_dom<PR, C, TS>;
  const size_t lds = lds_bytes(PR, C, TS);
  // idempotent; the call is cheap beside the launch
  MBBS_HIP(hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  const int grid = p.G == 1 ? p.units : p.ngroups * p.G;
  // one thread per (site, column chunk), per entry of the staged faces, and 16
  // per column for the domain sums (the most where a domain has few sites; lg is
  // at most 16, so TS holds them)
  const int thr = (std::max({p.T, p.H, 2 * (p.n[0] + p.n[1]), 2 * (p.n[2] + p.n[3]), 16 * p.lg}) + 63) / 64 * 64;
  MBBS_CHECK(thr <= TS, "domain solve: more threads than LDS cells per row");
  DomArgs a{};
  a.P = p;
  a.sy = sy;
  const Geom& g = lat->g;
  for (int m = 0; m < 4; ++m) {
    a.nd[m] = g.nd[m]; a.b[m] = g.b[m]; a.lstride[m] = lat->gk.lstride[m];
    a.ph[m][0] = g.ph[m][0]; a.ph[m][1] = g.ph[m][1];
  }
  a.ndomc = g.ndom / 2; a.nsys = lat->nsys; a.ndt = lat->gk.ndt; a.Vb = g.Vb; a.fstride = lat->gk.fstride;
  a.colour = colour; a.mode = mode; a.nmr = nmr;
  a.clov = lat->gk.clov; a.cinv64 = lat->gk.cinv64[DM]; a.cinv32 = lat->gk.cinv32[DM];
  a.kappa = lat->kappa; a.kap = lat->gk.kap;
  a.eta = b.eta; a.psi = b.psi; a.U = lat->Udp[PR]; a.frozen = frozen;
  hipLaunchKernelGGL(fn, dim3(grid), dim3(thr), lds, st, a);
  MBBS_HIP(hipGetLastError());
  return MBBS_OK;
}
template <int PR, int C>
int launch_dom(const mbbs_lattice_s* lat, const SapBuffers& b, const DomPlan& p, int colour, int mode, int nmr,
               const DomSync& sy, const int* frozen, hipStream_t st) {
  return p.TS == 256 ? launch_dom_ts<PR, C, 256>(lat, b, p, colour, mode, nmr, sy, frozen, st)
                     : launch_dom_ts<PR, C, 512>(lat, b, p, colour, mode, nmr, sy, frozen, st);
}

}  // namespace

// (All shapes that dom_plan considers.)  Links are addressed by 32-bit byte offsets.
bool dom_reads_links(const mbbs_lattice_s* lat, int prec) {
  const Geom& g = lat->g;
  if ((size_t)g.V * 4 * (prec == P64 ? 9 : 5) * 16 >= (1ull << 32)) return false;
  DomPlan p{};
  for (const int TS : {256, 512})
    for (int np = 1; np <= 8; np *= 2)
      if (pick_shape(g, np, TS, &p) && 8 * p.G <= lat->ncu && dom_pays(p, g.Vb, 1 << 30)) return true;
  return false;
}

bool dom_plan(const mbbs_lattice_s* lat, const SapBuffers& b, int nmr, DomPlan* out) {
  if (b.ssor || ((uintptr_t)b.eta | (uintptr_t)b.r | (uintptr_t)b.psi) & 15) return false;
  return dom_plan(lat, b.L, b.prec, nmr, (size_t)((char*)b.psi - (char*)b.r), out);
}

bool dom_plan(const mbbs_lattice_s* lat, int L, int prec, int nmr, size_t room, DomPlan* out) {
  if (lat->mr_fused >= 0) return false;   // the caller chose another form
  if (prec == P16 || !lat->Udp[prec]) return false;
  const Geom& g = lat->g;
  if (L > 64 || (nmr == 1 && g.Vb > 256)) return false;   // (the latter: no search for what dom_pays refuses)
  const int ncu = lat->ncu;
  // Two columns per thread in FP32 arithmetic (a link serves both) and the
  // largest tiles, unless a launch would then leave CUs without a workgroup.
  const int cmax = prec == P64 || L % 2 ? 1 : 2;
  // (counted for one system of a batch: a batch runs its systems as they run alone)
  DomPlan p{};
  size_t most = 0;
  auto consider = [&](int C, int TS) {
    if (most >= (size_t)ncu) return;
    DomPlan best{};
    bool have = false;
    for (int np = 1; np <= 8 && np * C <= std::min(L, 16); np *= 2) {
      if (L % (np * C)) continue;
      DomPlan q{};
      if (!pick_shape(g, np, TS, &q) || 8 * q.G > ncu) continue;
      q.np = np; q.C = C; q.lg = np * C; q.ncg = L / q.lg;
      q.units = g.ndom / 2 / lat->nsys * q.ncg;
      if (TS == 512 && q.G == 1) continue;   // TS = 256 holds two such workgroups per CU
      // a whole domain with more columns only while the chip stays full; tiles:
      // the fewest, then the smallest halo
      if (!have || (best.G == 1 ? q.G == 1 && q.units >= 2 * ncu : q.G < best.G || (q.G == best.G && q.H < best.H))) {
        best = q;
        have = true;
      }
    }
    if (have && (size_t)best.units * best.G > most) { p = best; most = (size_t)best.units * best.G; }
  };
  DomPlan whole{};
  const bool one = pick_shape(g, 1, 256, &whole) && whole.G == 1;
  for (int C = cmax; C >= 1; --C) {
    if (!one) consider(C, 512);
    consider(C, 256);
  }
  if (most == 0 || !dom_pays(p, g.Vb, nmr)) return false;
  p.units *= lat->nsys;
  p.ngroups = 1;
  if (p.G > 1) {
    // one workgroup per CU (TS = 512), else two; the groups' words and slots
    // lie in the fields r and w, which this path does not use otherwise
    const size_t slot = slot_bytes(p, prec);
    if (slot >= (1ull << 31)) return false;
    p.ngroups = std::min(p.units, (p.TS == 512 ? 1 : 2) * ncu / p.G);
    while (p.ngroups > 0 && al(sync_ints(p) * sizeof(int)) + p.ngroups * slot > room) --p.ngroups;
    if (p.ngroups < 1) return false;
  }
  *out = p;
  return true;
}

int dom_to(const mbbs_lattice_s* lat, int prec, int L, const DomPlan& p, const int* order, const double2* in,
           const double2* gam, void* out, unsigned* clear, int nclear, const int* frozen, hipStream_t st) {
  const Geom& g = lat->g;
  const int SB = conv_sites(g.Vb, L), nb = g.V / SB, thr = (SB * L + 63) / 64 * 64;
  const size_t shm = ((size_t)SB * 12 * L + (gam ? (size_t)L * L : 0)) * sizeof(double2);
  auto go = [&](auto fn, auto* o) {
    hipLaunchKernelGGL(fn, dim3(nb), dim3(thr), shm, st, lat->gk, p, L, SB, in, gam, o, clear, nclear, order, frozen);
  };
  if (prec == P64) {
    if (gam && L == 12) go(k_to_dom<P64, 12>, (double2*)out);
    else go(k_to_dom<P64>, (double2*)out);
  } else {
    if (gam && L == 12) go(k_to_dom<P32, 12>, (float2*)out);
    else go(k_to_dom<P32>, (float2*)out);
  }
  MBBS_HIP(hipGetLastError());
  return MBBS_OK;
}
int dom_from(const mbbs_lattice_s* lat, int prec, int L, const DomPlan& p, const int* order, const void* in,
             double2* out, const int* lost, const int* frozen, hipStream_t st) {
  const Geom& g = lat->g;
  const int SB = conv_sites(g.Vb, L), nb = g.V / SB, thr = (SB * L + 63) / 64 * 64;
  const size_t rows = (size_t)SB * 12 * L;
  if (prec == P64)
    hipLaunchKernelGGL(k_from_dom<double>, dim3(nb), dim3(thr), rows * 16, st, lat->gk, p, L, SB,
                       (const cplx<double>*)in, out, order, lost, frozen);
  else
    hipLaunchKernelGGL(k_from_dom<float>, dim3(nb), dim3(thr), rows * 8, st, lat->gk, p, L, SB, (const cplx<float>*)in,
                       out, order, lost, frozen);
  MBBS_HIP(hipGetLastError());
  return MBBS_OK;
}

int dom_sap_apply(const mbbs_lattice_s* lat, const SapBuffers& b, const DomPlan& p, int ncy, int nmr,
                  const double2* in, const double2* gam, double2* out, const int* frozen, hipStream_t st,
                  Profiler* prof) {
  const int nlaunch = 2 * ncy;
  const size_t nclear = p.G > 1 ? sync_ints(p) : 0;
  unsigned* clear = (unsigned*)b.r;
  if (prof) prof->begin(MBBS_K_CONVERT);
  MBBS_TRY(dom_to(lat, b.prec, b.L, p, nullptr, in, gam, b.eta, clear, (int)nclear, frozen, st));
  if (prof) prof->end();
  DomSync sy{};
  sy.step_polls = lat->sap_polls;
  if (p.G > 1) {
    sy.lost = (int*)clear + SYNC_LOST;
    sy.words = (u4*)(clear + SYNC_WORDS);
    sy.next = (unsigned long long*)(sy.words + (size_t)p.ngroups * 2 * p.G * 3 * p.lg);
    sy.flags = sy.next + p.ngroups;
    sy.slots = (char*)b.r + al(nclear * sizeof(int));
    sy.slot_bytes = slot_bytes(p, b.prec);
  }
  for (int l = 0; l < nlaunch; ++l) {
    const int colour = l & 1, mode = l >= 2 ? 2 : l;
    sy.counters = (int*)clear + (l & 1) * 2;
    sy.counters_next = (int*)clear + (~l & 1) * 2;
    sy.tag0 = (unsigned)l * ((unsigned)p.units * (2u * nmr + 2) + 4);
    if (prof) prof->begin(MBBS_K_MR_DSLASH);
    const int rc = b.prec == P64 ? launch_dom<P64, 1>(lat, b, p, colour, mode, nmr, sy, frozen, st)
                   : p.C == 2    ? launch_dom<P32, 2>(lat, b, p, colour, mode, nmr, sy, frozen, st)
                                 : launch_dom<P32, 1>(lat, b, p, colour, mode, nmr, sy, frozen, st);
    MBBS_TRY(rc);
    if (prof) prof->end();
  }
  if (prof) prof->begin(MBBS_K_CONVERT);
  MBBS_TRY(dom_from(lat, b.prec, b.L, p, nullptr, b.psi, out, sy.lost, frozen, st));
  if (prof) prof->end();
  return MBBS_OK;
}

}  // namespace mbbs
