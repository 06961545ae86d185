// Semi-implicit scheme: the slice force f1(A, B) of every link in one pass (Sec. 3, fig. wilson;
// the potential between two time slices and the derivative rule are stated in semi.hip).
//
// A wavefront owns a column of whole x rows of a layer (8 <= nt <= 64: 64 / nt of them, x
// neighbours in other lanes) and marches along z through a
// chunk of layers.  At each layer it forms the plaquette-like loops based at its sites
// once and hands each loop's derivative to the links that carry it:
//   * links of its own site: accumulated directly;
//   * links at x + e_x (factor 1 of an (x, y) or (x, z) loop): pulled by the next lane;
//   * links at x + e_z (factor 2 of an (x, z) or (y, z) loop): carried to the next layer;
//   * links at x + e_y (factor 2 of an (x, y) loop, factor 1 of a (y, z) loop): the site
//     above forms those loops again at its base - e_y (another wavefront's column).
// Per site and layer 30 links are loaded (MODE = 1: 26 and two cached loops; about 150 when every link
// forms all its loops), and 42 matrix products, 16 derivatives of a loop and 10 transports are formed
// (MODE = 1).  With MODE = 1 the pass also completes the fixed-point iteration of each link as soon as its
// force is complete (E' = Ebase + dt f1, under-relaxed, new trial link), so the force is
// never stored; MODE = 0 stores f1 (the per-step term f1(U(t), U(t - dt))).
#include <algorithm>
#include "internal.h"
#include "stencil.h"

namespace gl {

namespace {

// Products of the march.  SU(2): each component one chain of fused multiply-adds, the largest product
// last: links are near 1, so the terms without the zeroth component are small, and with them first
// single precision leaves 0.70 of the error in E that the compiler's own choice of fused terms leaves
// per direction (semi.hip), the other way round 1.2.
template <typename G> struct MarchOps : G {};
template <typename T> struct MarchOps<Su2<T>> : Su2<T> {
  using L = Q2<T>;
  using A = Alg2<T>;
  // component k > 0 of a b: a0 b_k + a_k b0 - (a x b)_k
  static __device__ __forceinline__ T vec(const L& a, const L& b, int k, int i, int j) {
    return fmx(a.q[0], b.q[k], fmx(a.q[k], b.q[0], -fmx(a.q[i], b.q[j], -(a.q[j] * b.q[i]))));
  }
  static __device__ __forceinline__ L mul(const L& a, const L& b) {
    L r;
    r.q[0] = fmx(a.q[0], b.q[0], -fmx(a.q[1], b.q[1], fmx(a.q[2], b.q[2], a.q[3] * b.q[3])));
    r.q[1] = vec(a, b, 1, 2, 3);
    r.q[2] = vec(a, b, 2, 3, 1);
    r.q[3] = vec(a, b, 3, 1, 2);
    return r;
  }
  static __device__ __forceinline__ L mul_dag(const L& a, const L& b) { return mul(a, Su2<T>::dag(b)); }
  static __device__ __forceinline__ A proj_mul_dag(const L& a, const L& b) {
    const L c = Su2<T>::dag(b);
    A r;
    r.c[0] = 2 * vec(a, c, 1, 2, 3);
    r.c[1] = 2 * vec(a, c, 2, 3, 1);
    r.c[2] = 2 * vec(a, c, 3, 1, 2);
    return r;
  }
  static __device__ __forceinline__ A transport(const L& u, const A& x) {
    return Su2<T>::link_as_alg(mul(mul(Su2<T>::dag(u), Su2<T>::alg_as_link(x)), u));
  }
};

// components of M + M^dag (hermitian; its traceless part)
template <typename G> __device__ __forceinline__ typename G::Alg hsum(const typename G::Link& m) {
  typename G::Link h = m;
  G::add_to(h, G::dag(m), (typename G::Real)(G::NC == 3 ? 1 : -1));
  return G::alg_from_herm(h);
}
template <typename A, typename R> __device__ __forceinline__ void axpy(A& acc, R s, const A& x) {
  constexpr int NG = sizeof(acc.c) / sizeof(acc.c[0]);
#pragma unroll
  for (int k = 0; k < NG; ++k) acc.c[k] = fmx(s, x.c[k], acc.c[k]);
}
// Components of H = M + M^dag for M = C Y (LEFT = false) or M = Y C (LEFT = true), with Y the
// hermitian matrix of the algebra element y, without forming M: only the 15 entries of M
// that H's traceless part reads, and Y's real diagonal taken as real (a general product
// would multiply its zero imaginary parts too).  SU(3); SU(2) takes the general route.
template <bool LEFT, typename R>
__device__ __forceinline__ Alg3<R> hs_herm(const M3<R>& C, const Alg3<R>& y) {
  const typename Su3<R>::Herm q = Su3<R>::herm_c(y, R(1));
  // Y_kj = (yr, yi)
  auto Y = [&](int k, int j, R& yr, R& yi) {
    if (k == j) { yr = q.d[j]; yi = R(0); return; }
    const int n = (k == 0 || j == 0) ? ((k == 1 || j == 1) ? 0 : 1) : 2;
    yr = q.r[n];
    yi = k < j ? q.i[n] : -q.i[n];
  };
  // entry (p, j) of M, real (want_im false) or imaginary part
  auto ent = [&](int p, int j, bool want_im) -> R {
    R acc = R(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      R yr, yi;
      R cr, ci;
      if (LEFT) {   // M_pj = sum_k Y_pk C_kj
        Y(p, k, yr, yi);
        cr = C.re[k][j];
        ci = C.im[k][j];
        const bool real_y = p == k;
        if (!want_im) {
          acc = fmx(yr, cr, acc);
          if (!real_y) acc = fmx(-yi, ci, acc);
        } else {
          acc = fmx(yr, ci, acc);
          if (!real_y) acc = fmx(yi, cr, acc);
        }
      } else {      // M_pj = sum_k C_pk Y_kj
        Y(k, j, yr, yi);
        cr = C.re[p][k];
        ci = C.im[p][k];
        const bool real_y = k == j;
        if (!want_im) {
          acc = fmx(cr, yr, acc);
          if (!real_y) acc = fmx(-ci, yi, acc);
        } else {
          acc = fmx(ci, yr, acc);
          if (!real_y) acc = fmx(cr, yi, acc);
        }
      }
    }
    return acc;
  };
  const R is3 = R(0.57735026918962576451);
  const R m00 = ent(0, 0, false), m11 = ent(1, 1, false), m22 = ent(2, 2, false);
  Alg3<R> r;
  r.c[0] = R(2) * (ent(0, 1, false) + ent(1, 0, false));
  r.c[1] = R(2) * (ent(1, 0, true) - ent(0, 1, true));
  r.c[2] = R(2) * (m00 - m11);
  r.c[3] = R(2) * (ent(0, 2, false) + ent(2, 0, false));
  r.c[4] = R(2) * (ent(2, 0, true) - ent(0, 2, true));
  r.c[5] = R(2) * (ent(1, 2, false) + ent(2, 1, false));
  r.c[6] = R(2) * (ent(2, 1, true) - ent(1, 2, true));
  r.c[7] = R(2) * (m00 + m11 - R(2) * m22) * is3;
  return r;
}
template <bool LEFT, typename R>
__device__ __forceinline__ Alg2<R> hs_herm(const Q2<R>& C, const Alg2<R>& y) {
  using G = MarchOps<Su2<R>>;
  const Q2<R> Y = G::herm_from_alg(y);
  return hsum<G>(LEFT ? G::mul(Y, C) : G::mul(C, Y));
}

// Algebra element in a per-thread slot of the work-group's LDS (a thread only touches its
// own slot, so no barrier is needed): components k at p[k * BS].
template <int BS, typename Ag, typename R> struct AccL {
  R* p;
  static constexpr int NG = sizeof(Ag::c) / sizeof(R);
  __device__ __forceinline__ Ag get() const {
    Ag v;
#pragma unroll
    for (int k = 0; k < NG; ++k) v.c[k] = p[k * BS];
    return v;
  }
  __device__ __forceinline__ void set(const Ag& x) {
#pragma unroll
    for (int k = 0; k < NG; ++k) p[k * BS] = x.c[k];
  }
  __device__ __forceinline__ void add(R s, const Ag& x) {
#pragma unroll
    for (int k = 0; k < NG; ++k) p[k * BS] = fmx(s, x.c[k], p[k * BS]);
  }
};
template <typename R> __device__ __forceinline__ R link_token(const M3<R>& m) { return m.re[2][2]; }
template <typename R> __device__ __forceinline__ R link_token(const Q2<R>& m) { return m.q[3]; }

}  // namespace

constexpr int MARCH_BS = 256;
// stages of a layer, and of the layer before a chunk (its carries)
constexpr int MARCH_SUB = 4, MARCH_WARM = 2;
// What lives across the stages sits in per-thread LDS slots: the derivatives of the site's x
// and y links, which double as the carries to the next layer (2 n_g reals), and the site's z
// links of both slices, loaded once per layer (2 stored links): 80 KB per work-group for
// SU(3) in double precision, two work-groups per CU at two waves per SIMD.
//
// What bounds it: vector memory.  The columns that march at once hold about 30 MB per XCD
// against 4 MB of L2, so a link that is loaded again in a later stage comes from beyond the L2.
// So each stage forms every loop of a plane and loads each link it needs once, but for the z link at y + 1
// of slice B (stage 2) and, in MODE 0, the site's x link of slice A (stage 0), loaded twice to save
// registers: an iteration loads 26 links, two loops and the field and guess per site and layer, 3.2 KB
// for SU(3) FP64, and stores 0.5 KB, at 6.6 TB/s.  With one loop per micro-step (21 of them, 55 links and
// 5 cached loops, 6.4 KB) an iteration at 512 x 64 x 64 took 1.51 ms, now 1.16 ms (1.13 ms with the loops
// cut to two rows), and the per-step force 1.53 ms, now 0.92 ms (medians over a solve's launches).
// Registers: a link is held as stored (24 registers instead of 36) and rebuilt at each use,
// scheduling fences keep the products of a stage apart, projections are formed from the loops
// where they are used, and loads take a uniform base and a 32-bit offset.  Without each of
// these the kernel spilled 100-300 registers (34 are left in MODE 1, 39 with the general record offsets).

// MarchIter (internal.h): Ebase = E(t - dt/2) + dt f1(U(t), U(t - dt)) (+ dt j on z links);
// Et the iterate E(t + dt/2), updated in place; Ut_out the new trial links exp(i a dt E') U(t);
// conv = [max |E' - E_old|, max |E'|] of this iteration (atomic max); F the MODE 0 output;
// cache: the loops C_xy of slice A alone based at each site, which MODE 0 stores (it forms them
// anyway) and the iterations of the step read back (A = U(t) is fixed for the step).  Whole matrices:
// links are special unitary only up to their storage's rounding, and a third row rebuilt from two
// leaves the loop's a quarter to a half further off.  The (x, z) and (y, z) loops of A alone are
// formed from the links that their stage loads anyway.

// Rows of 8 to 64 sites.  A row that leaves lanes idle (33: 31 of 64) still pays: two steps of 2.1 million
// sites at dt = a_L took 83-89 ms with a kernel per link direction (semi.hip) and take 59 ms at nt =
// 33, 47-50 ms at 45 and 48, 42 ms at 28 (38 ms at 64).
bool march_geometry(const Geom& g) { return g.nt >= 8 && g.nt <= 64; }
size_t march_cache_elems(const Geom& g, int nc) { return (size_t)(nc == 3 ? 18 : 4) * g.Vp; }

__device__ __forceinline__ void atomic_max_nn(double* addr, double v) {
  atomicMax((unsigned long long*)addr, (unsigned long long)__double_as_longlong(v));
}

// AL: layers are whole records (nt^2 a multiple of 64), so an offset only depends on (x, y) and is
// formed once; with the general form everywhere 512 x 64 x 64 took 2.7% longer.
template <typename G, typename T, int MODE, bool AL>
__global__ void __launch_bounds__(MARCH_BS) __attribute__((amdgpu_waves_per_eu(2))) k_semi_march(const T* __restrict__ A, const T* __restrict__ B, Geom g,
                                                         MarchIter it, int ncg, int nch, int lz) {
  using L = typename G::Link;
  using M = MarchOps<G>;
  using Ag = typename G::Alg;
  using R = typename G::Real;
  constexpr int NG = G::NG;
  if constexpr (MODE == 1) {
    if (it.conv_prev) {
      const double e = it.conv_prev[1];
      if (it.conv_prev[0] <= it.tol * (e > 0.0 ? e : 1e-300)) return;   // converged before
    }
  }
  const int64_t Vp = g.Vp;
  // work-group -> (chunk, column group), XCD-contiguous so that neighbouring column groups
  // (the y halo rows) of one chunk share an L2
  const uint32_t nb = (uint32_t)(ncg * nch);
  const uint32_t bid = xcd_remap(blockIdx.x, nb);
  const int cg = (int)(bid % (uint32_t)ncg), ch = (int)(bid / (uint32_t)ncg);
  const int col = cg * (MARCH_BS / 64) + (int)(threadIdx.x >> 6);
  const int rpw = 64 / g.nt;   // rows per wavefront
  if (col * rpw >= g.nt || ch >= nch) return;   // uniform over the wavefront
  const int lane = (int)(threadIdx.x & 63u);
  // a lane without a site of its own does the first lane's work (the same loads, pulls and
  // stores of the same values): no store is masked, which would split the stages' blocks
  const int as = lane < rpw * g.nt && col * rpw + lane / g.nt < g.nt ? lane : 0;
  Site b0;
  b0.x = as % g.nt;
  b0.y = col * rpw + as / g.nt;
  const int z0 = ch * lz;
  const int z1 = min(z0 + lz, g.nz);
  XNbr xn;
  xn.ap = 4 * (as + (b0.x + 1 < g.nt ? 1 : 1 - g.nt));
  xn.am = 4 * (as + (b0.x > 0 ? -1 : g.nt - 1));
  // Every load goes through an empty asm statement on its offset that also takes a token, a
  // value of a loop product already formed: the compiler cannot merge it with an earlier load
  // of the same link and cannot issue it before that product exists (hoisting the loads
  // of later loops to the top of a stage would hold their links live all along).
  R tok = R(0);
  // Links are addressed by a uniform base (direction, and the record in which the layer starts)
  // plus a 32-bit offset from there.
  constexpr int SW = StoredWidth<L>::value;
  constexpr uint32_t RBYTES = RecShape<T, SW>::BYTES;
  const uint64_t dir_bytes = (uint64_t)Vp * SW * sizeof(T);
  // offset of in-layer index q where the layer's first site is site ph of its record
  auto in_layer = [](uint32_t q, uint32_t ph) __attribute__((always_inline)) {
    return ((q + ph) / RB) * RBYTES + ((q + ph) % RB) * 16;
  };
  // the site and its +y and -y neighbours in the layer: index, or (AL) offset
  const uint32_t t = (uint32_t)(b0.y * g.nt + b0.x);
  auto place = [&](uint32_t q) __attribute__((always_inline)) { return AL ? in_layer(q, 0) : q; };
  const uint32_t o_t = place(t), o_py = place((uint32_t)(wrap_add(b0.y, 1, g.nt) * g.nt + b0.x)),
                 o_my = place((uint32_t)(wrap_add(b0.y, -1, g.nt) * g.nt + b0.x));
  struct Layer {   // its first record's offset in a direction, and its first site's place there
    uint64_t rec;
    uint32_t ph;
  };
  auto layer_at = [&](int z) __attribute__((always_inline)) {
    const uint32_t s0 = (uint32_t)z * (uint32_t)g.layer;
    return Layer{(uint64_t)(s0 / RB) * RBYTES, AL ? 0u : s0 % RB};
  };
  struct Raw {   // a link as stored (SU(3): two rows); full() rebuilds it at each use
    R v[SW];
  };
  auto ld = [&](Raw& l, const T* U, int d, const Layer& y, uint32_t q) __attribute__((always_inline)) {
    uint32_t off = AL ? q : in_layer(q, y.ph);
    asm volatile("" : "+v"(off) : "v"(tok));
    using NV = typename NVec16<T>::type;
    const char* base = (const char*)U + (uint64_t)d * dir_bytes + y.rec;
#pragma unroll
    for (int q = 0; q < SW * (int)sizeof(T) / 16; ++q) {
      const NV x = *(const NV*)(base + q * (RB * 16) + off);
#pragma unroll
      for (int k = 0; k < 16 / (int)sizeof(T); ++k) l.v[q * (16 / (int)sizeof(T)) + k] = (R)x[k];
    }
  };
  // the cached loop based at in-layer index q of layer z
  auto ld_loop = [&](L& m, int z, uint32_t q) __attribute__((always_inline)) {
    asm volatile("" : "+v"(q) : "v"(tok));
    constexpr int CW = FullWidth<L>::value;
    R v[CW];
    load_comps<R, T, CW>(v, (const T*)it.cache, (uint32_t)z * (uint32_t)g.layer + q);
#pragma unroll
    for (int k = 0; k < CW; ++k) full_real(m, k) = v[k];
  };
  auto keep_loop = [&](L& m, uint32_t s) __attribute__((always_inline)) {
    constexpr int CW = FullWidth<L>::value;
    R v[CW];
#pragma unroll
    for (int k = 0; k < CW; ++k) v[k] = full_real(m, k);
    store_comps<R, T, CW>(v, (T*)it.cache, s);
  };
  auto full = [&](Raw& r) __attribute__((always_inline)) -> L {
#pragma unroll
    for (int k = 0; k < SW / 2; ++k) asm volatile("" : "+v"(r.v[k]));   // no third row kept from an earlier use
    L l;
    link_from_stored(l, r.v);
    return l;
  };
  auto pulled = [&](const Raw& r) __attribute__((always_inline)) -> L {   // of the lane at x + e_x
    Raw p;
#pragma unroll
    for (int k = 0; k < SW; ++k) p.v[k] = lane_pull(r.v[k], xn.ap);
    L l;
    link_from_stored(l, p.v);
    return l;
  };
  // the z links of the site on both slices, loaded once per layer into per-thread LDS slots of
  // 16-byte chunks: zl(k) rebuilds slice k's (0 A, 1 B), zlx(k) that of the lane at x + e_x
  using V16 = typename Vec16<T>::type;
  constexpr int NCH = SW * (int)sizeof(T) / 16, VW = 16 / (int)sizeof(T);
  __shared__ V16 zpark[2 * NCH * MARCH_BS];
  auto park = [&](const Raw& r, int k) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      V16 x;
      T* e = (T*)&x;
#pragma unroll
      for (int j = 0; j < VW; ++j) e[j] = (T)r.v[q * VW + j];
      zpark[(k * NCH + q) * MARCH_BS + threadIdx.x] = x;
    }
  };
  auto unpark = [&](uint32_t slot, int k) __attribute__((always_inline)) -> L {
    asm volatile("" : "+v"(slot));   // read again at each use
    R v[SW];
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      const V16 x = zpark[(k * NCH + q) * MARCH_BS + slot];
      const T* e = (const T*)&x;
#pragma unroll
      for (int j = 0; j < VW; ++j) v[q * VW + j] = (R)e[j];
    }
    L l;
    link_from_stored(l, v);
    return l;
  };
  const uint32_t slot_x = (threadIdx.x & ~63u) + (uint32_t)(xn.ap >> 2);   // of the lane at x + e_x
  auto zl = [&](int k) __attribute__((always_inline)) -> L { return unpark(threadIdx.x, k); };
  auto zlx = [&](int k) __attribute__((always_inline)) -> L { return unpark(slot_x, k); };
  auto fence = []() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
  double dmax = 0.0, emax = 0.0;
  bool bad = false;
  // finish link d of site s with its complete derivative acc (dv/dX as components); u() = U_d(s)
  // on slice A
  auto finish = [&](const Ag& acc, int d, uint32_t s, auto&& u) __attribute__((always_inline)) {
    if constexpr (MODE == 0) {
      Ag f;
#pragma unroll
      for (int k = 0; k < NG; ++k) f.c[k] = (R)it.ma[d] * acc.c[k];
      store_alg(f, (T*)it.F, d, s, Vp);
    } else {
      Ag e, eo;
      load_alg_own(e, (const T*)it.Ebase, d, s, Vp);
      load_alg_own(eo, (const T*)it.Et, d, s, Vp);
      const R om = (R)it.omega;
#pragma unroll
      for (int k = 0; k < NG; ++k) {
        const R en = fmx((R)it.madt[d], acc.c[k], e.c[k]);
        dmax = fmax(dmax, fabs((double)en - (double)eo.c[k]));
        emax = fmax(emax, fabs((double)en));
        bad |= !isfinite((double)en);
        e.c[k] = fmx(om, en - eo.c[k], eo.c[k]);
      }
      store_alg(e, (T*)it.Et, d, s, Vp);
      const L w = G::expi(e, (R)-it.madt[d]);
      fence();
      store_link(M::mul(w, u()), (T*)it.Ut_out, d, s, Vp);
    }
  };
  // The work of a layer is a sequence of four stages, each its own basic block (a loop that is
  // not unrolled over a switch on a uniform stage number), so only the accumulators live across
  // them.  A stage loads each link it needs once; the token orders the loads of its second half
  // behind the loops of its first.
  //   fx, fy, fz: derivative of the site's x, y, z links; cx, cy: carries to the x, y links
  //   of the next layer; snd: the (x, z) loops' derivative for the z link at s + e_x, pulled by
  //   the next lane.
  // Stages 1 and 2 also serve the warm-up (the carries from the layer before the chunk),
  // where their other outputs are discarded.
  // fx doubles as the carry to the x link of the next layer (from the end of stage 1 on), fy as
  // that to the y link: the derivative is complete when the next carry is
  __shared__ R acc_lds[2 * NG * MARCH_BS];
  using A_ = AccL<MARCH_BS, Ag, R>;
  A_ fx{acc_lds + threadIdx.x}, fy{acc_lds + NG * MARCH_BS + threadIdx.x};
  fx.set(G::alg_zero());
  fy.set(G::alg_zero());
  Ag fz = G::alg_zero();
  constexpr int NSUB = MARCH_SUB, NWARM = MARCH_WARM;
  const int zm = z0 > 0 ? z0 - 1 : g.nz - 1;
  const int nq = NWARM + (z1 - z0) * NSUB;
#pragma unroll 1
  for (int q = 0; q < nq; ++q) {
    const bool warm = q < NWARM;
    const int z = warm ? zm : z0 + (q - NWARM) / NSUB;
    const int stage = warm ? 1 + q : (q - NWARM) % NSUB;
    const int zp = z + 1 < g.nz ? z + 1 : 0;
    const Layer ly = layer_at(z), lyp = layer_at(zp);
    const uint32_t site_z = (uint32_t)z * (uint32_t)g.layer + t;   // site index (E, Et, outputs)
    switch (stage) {
      // ---- (x, y) plane at the base: x link factor 0, y link factor 3, y link at s + e_x factor
      // 1; then at base - e_y, where the x link is factor 2 (daggered), W = C F3
      case 0: {
        Raw u, v, w;
        L m;
        ld(u, B, 0, ly, o_t);
        ld(v, B, 1, ly, o_t);
        ld(w, B, 0, ly, o_py);
        m = M::mul(full(u), pulled(v));
        fence();
        m = M::mul_dag(m, full(w));
        fence();
        Ag P = M::proj_mul_dag(m, full(v));
        tok = P.c[0];
        fence();
        // the loop of slice A alone: MODE 0 forms and stores it, MODE 1 reads it back
        if constexpr (MODE == 0) {
          Raw x;
          ld(x, A, 0, ly, o_t);
          ld(v, A, 1, ly, o_t);
          ld(w, A, 0, ly, o_py);
          m = M::mul(full(x), pulled(v));
          fence();
          m = M::mul_dag(m, full(w));
          fence();
          m = M::mul_dag(m, full(v));
          keep_loop(m, site_z);
          v = x;
        } else {
          ld_loop(m, z, t);
          ld(v, A, 0, ly, o_t);
        }
        fence();
        Ag fv = fx.get();   // the carry
        const Ag hf = hs_herm<false>(m, P);
        axpy(fv, (R)it.k[0], hf);
        Ag gv = fy.get();
        axpy(gv, (R)-it.k[0], hs_herm<true>(m, P));
        fence();
        axpy(gv, (R)it.k[0], pull_alg(M::transport(full(v), hf), xn.am));
        fy.set(gv);
        tok = gv.c[0];
        fence();
        ld(w, B, 0, ly, o_my);
        ld(v, B, 1, ly, o_my);
        m = M::mul(full(w), pulled(v));
        fence();
        m = M::mul_dag(m, full(u));
        fence();
        P = M::proj_mul_dag(m, full(v));
        tok = P.c[0];
        fence();
        if constexpr (MODE == 0) {
          ld(u, A, 0, ly, o_my);
          ld(v, A, 1, ly, o_my);
          ld(w, A, 0, ly, o_t);
          m = M::mul(full(u), pulled(v));
          fence();
          m = M::mul_dag(m, full(w));
          fence();
          m = M::mul_dag(m, full(v));
        } else {
          ld_loop(m, z, (uint32_t)(wrap_add(b0.y, -1, g.nt) * g.nt + b0.x));
          ld(v, A, 1, ly, o_my);
        }
        fence();
        const Ag hb = hs_herm<true>(m, P);
        fence();
        axpy(fv, (R)-it.k[0], M::transport(full(v), hb));
        fx.set(fv);
        tok = fv.c[0];
        break;
      }
      // ---- (x, z) plane at the base: x link factor 0, z link factor 3, x link at s + e_z
      // factor 2 (carry), z link at s + e_x factor 1 (snd)
      case 1: {
        Raw a0, u;
        L ca, cb;
        {
          Raw b2, a2;
          ld(b2, B, 2, ly, o_t);
          ld(a2, A, 2, ly, o_t);
          ld(a0, A, 0, ly, o_t);
          ld(u, A, 0, lyp, o_t);
          park(a2, 0);
          park(b2, 1);
        }
        // the wavefront's own writes before its other lanes' reads
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        cb = M::mul(full(a0), zlx(1));
        fence();
        cb = M::mul_dag(cb, full(u));
        fence();
        cb = M::mul_dag(cb, zl(1));
        fence();
        ca = M::mul(full(a0), zlx(0));
        fence();
        ca = M::mul_dag(ca, full(u));
        fence();
        ca = M::mul_dag(ca, zl(0));
        fence();
        if (!warm) {
          Ag hf = hs_herm<false>(ca, G::proj(cb));
          fx.add((R)it.k[1], hf);
          fence();
          hf = M::transport(full(a0), hf);   // on the z link at s + e_x
          fence();
          fz = pull_alg(hf, xn.am);
          hf = hs_herm<false>(cb, G::proj(ca));
          fx.add((R)it.k[1], hf);
          fence();
        }
        Ag cv = hs_herm<true>(ca, G::proj(cb));
        axpy(fz, R(-1), cv);
        fence();
        cv = M::transport(zl(0), cv);
        fence();
        {
          const Ag hb = hs_herm<true>(cb, G::proj(ca));
          fence();
          axpy(cv, R(1), M::transport(zl(1), hb));
        }
        fence();
#pragma unroll
        for (int k = 0; k < NG; ++k) cv.c[k] *= (R)-it.k[1];
        const Ag fv = fx.get();
        fx.set(cv);   // from here on the carry to the next layer
        tok = cv.c[0];
        if (warm) break;
        finish(fv, 0, site_z, [&]() { return full(a0); });   // the x link is complete
        fence();
        ld(u, B, 0, ly, o_t);
        ld(a0, B, 0, lyp, o_t);
        cb = M::mul(full(u), zlx(1));
        fence();
        cb = M::mul_dag(cb, full(a0));
        fence();
        const Ag P = M::proj_mul_dag(cb, zl(1));
        fence();
        ca = M::mul(full(u), zlx(0));
        fence();
        ca = M::mul_dag(ca, full(a0));
        fence();
        ca = M::mul_dag(ca, zl(0));
        fence();
        axpy(fz, R(-1), hs_herm<true>(ca, P));
        fence();
        {
          const Ag hf = hs_herm<false>(ca, P);
          fence();
          axpy(fz, R(1), pull_alg(M::transport(full(u), hf), xn.am));
        }
#pragma unroll
        for (int k = 0; k < NG; ++k) fz.c[k] *= (R)it.k[1];
        tok = fz.c[0];
        break;
      }
      // ---- (y, z) plane at the base: y link factor 0, z link factor 3, y link at s + e_z
      // factor 2 (carry); its factor 1 (z link at s + e_y) is formed by the site above
      case 2: {
        Raw a1, u, v;
        L ca, cb;
        ld(a1, A, 1, ly, o_t);
        ld(v, B, 2, ly, o_py);
        ld(u, A, 1, lyp, o_t);
        cb = M::mul(full(a1), full(v));
        tok = link_token(cb);
        fence();
        ld(v, A, 2, ly, o_py);
        cb = M::mul_dag(cb, full(u));
        fence();
        cb = M::mul_dag(cb, zl(1));
        fence();
        ca = M::mul(full(a1), full(v));
        fence();
        ca = M::mul_dag(ca, full(u));
        fence();
        ca = M::mul_dag(ca, zl(0));
        fence();
        if (!warm) {
          fy.add((R)it.k[2], hs_herm<false>(ca, G::proj(cb)));
          fence();
          fy.add((R)it.k[2], hs_herm<false>(cb, G::proj(ca)));
          fence();
        }
        Ag cv = hs_herm<true>(ca, G::proj(cb));
        axpy(fz, (R)-it.k[2], cv);
        fence();
        cv = M::transport(zl(0), cv);
        fence();
        {
          const Ag hb = hs_herm<true>(cb, G::proj(ca));
          fence();
          axpy(cv, R(1), M::transport(zl(1), hb));
        }
        fence();
#pragma unroll
        for (int k = 0; k < NG; ++k) cv.c[k] *= (R)-it.k[2];
        const Ag fv = fy.get();
        fy.set(cv);   // from here on the carry to the next layer
        tok = cv.c[0];
        if (warm) break;
        finish(fv, 1, site_z, [&]() { return full(a1); });   // the y link is complete
        fence();
        ld(u, B, 1, ly, o_t);
        ld(a1, B, 1, lyp, o_t);
        {
          Raw w;
          ld(w, B, 2, ly, o_py);
          cb = M::mul(full(u), full(w));
        }
        fence();
        cb = M::mul_dag(cb, full(a1));
        fence();
        const Ag P = M::proj_mul_dag(cb, zl(1));
        fence();
        ca = M::mul(full(u), full(v));
        fence();
        ca = M::mul_dag(ca, full(a1));
        fence();
        ca = M::mul_dag(ca, zl(0));
        fence();
        const Ag hb = hs_herm<true>(ca, P);
        axpy(fz, (R)-it.k[2], hb);
        tok = hb.c[0];
        break;
      }
      // ---- (y, z) plane at base - e_y: the z link is its factor 1, W = F0 (the y link at s - e_y)
      default: {
        Raw f0, f2, v, w;
        L m;
        ld(f0, A, 1, ly, o_my);
        ld(f2, A, 1, lyp, o_my);
        ld(w, B, 2, ly, o_my);
        m = M::mul(full(f0), zl(1));
        fence();
        m = M::mul_dag(m, full(f2));
        tok = link_token(m);
        fence();
        ld(v, A, 2, ly, o_my);
        Ag P = M::proj_mul_dag(m, full(w));
        fence();
        m = M::mul(full(f0), zl(0));
        fence();
        m = M::mul_dag(m, full(f2));
        fence();
        m = M::mul_dag(m, full(v));
        tok = link_token(m);
        fence();
        Raw g0;
        ld(g0, B, 1, ly, o_my);
        ld(f2, B, 1, lyp, o_my);
        {
          const Ag hf = hs_herm<false>(m, P);
          fence();
          axpy(fz, (R)it.k[2], M::transport(full(f0), hf));
        }
        fence();
        m = M::mul(full(g0), zl(1));
        fence();
        m = M::mul_dag(m, full(f2));
        fence();
        P = M::proj_mul_dag(m, full(w));
        fence();
        m = M::mul(full(g0), zl(0));
        fence();
        m = M::mul_dag(m, full(f2));
        fence();
        m = M::mul_dag(m, full(v));
        fence();
        {
          const Ag hf = hs_herm<false>(m, P);
          fence();
          axpy(fz, (R)it.k[2], M::transport(full(g0), hf));
        }
        tok = fz.c[0];
        fence();
        finish(fz, 2, site_z, [&]() { return zl(0); });   // the z link is complete
        break;
      }
    }
  }
  if constexpr (MODE == 1) {
    if (bad) dmax = INFINITY;
    for (int o = 32; o > 0; o >>= 1) {
      dmax = fmax(dmax, __shfl_down(dmax, o, 64));
      emax = fmax(emax, __shfl_down(emax, o, 64));
    }
    if (lane == 0) {
      atomic_max_nn(it.conv, dmax);
      atomic_max_nn(it.conv + 1, emax);
    }
  }
}

// Layers per chunk of the march.  A chunk first repeats the loops of the layer before it that
// feed its carries (MARCH_WARM of the MARCH_SUB stages of a layer), and a wavefront does
// its stages one after the other, so a launch takes (MARCH_WARM + lz MARCH_SUB) stages
// for every round of work-groups that the chip holds at once.  The length with the fewest is
// taken (the longest of equals: less repeated work): 16 layers on 512 x 64 x 64, which fill
// the chip in one round (8 layers, two rounds: 7% slower), down to single layers where the
// lattice is too small to fill it: 96 x 32 x 32 FP64, 24 work-groups of 16 layers 0.595 ms per
// iteration, 384 of one layer 0.109 ms (0.089 ms with four stages per layer).  The result does not depend on the length
// (the repeated loops are the same operations on the same links).
constexpr int MARCH_LZ_MAX = 16;
inline int march_chunk(int ncg, int nz, int resident) {
  int best = 1;
  int64_t best_cost = INT64_MAX;
  for (int lz = 1; lz <= MARCH_LZ_MAX; ++lz) {
    const int64_t groups = (int64_t)ncg * ((nz + lz - 1) / lz);
    const int64_t cost = (groups + resident - 1) / resident * (MARCH_WARM + (int64_t)std::min(lz, nz) * MARCH_SUB);
    if (cost <= best_cost) { best_cost = cost; best = lz; }
  }
  return best;
}

template <typename G, typename T>
void launch_semi_march(const T* A, const T* B, const Geom& g, const StepConst& c, int mode, const MarchIter& it_,
                       hipStream_t st) {
  const int rpw = 64 / g.nt, ncol = (g.nt + rpw - 1) / rpw;
  const int ncg = (ncol + MARCH_BS / 64 - 1) / (MARCH_BS / 64);
  MarchIter it = it_;
  it.k[0] = 0.25 / (c.a[0] * c.a[0] * c.a[1] * c.a[1]);
  it.k[1] = 0.125 / (c.a[0] * c.a[0] * c.a[2] * c.a[2]);
  it.k[2] = 0.125 / (c.a[1] * c.a[1] * c.a[2] * c.a[2]);
  for (int d = 0; d < 3; ++d) {
    it.ma[d] = -c.a[d];
    it.madt[d] = -c.a[d] * c.dt;
  }
  // work-groups at once on 256 CUs: 2 per CU for SU(3) in double precision and 3 in single, from the
  // kernel's registers; SU(2) 3 and 5, one less than its registers allow (4 in double: two steps of
  // 200 x 64 x 64 5.43 ms for 4.43, 200 x 33 x 33 3.11 for 2.75)
  constexpr int per_cu = sizeof(T) == 8 ? (G::NC == 3 ? 2 : 3) : (G::NC == 3 ? 3 : 5);
  const int lz = march_chunk(ncg, g.nz, per_cu * 256);
  const int nch = (g.nz + lz - 1) / lz;
  const dim3 grid((unsigned)(ncg * nch));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(MARCH_BS), 0, st, A, B, g, it, ncg, nch, lz);
  };
  if (g.layer % RB == 0) mode == 0 ? go(k_semi_march<G, T, 0, true>) : go(k_semi_march<G, T, 1, true>);
  else mode == 0 ? go(k_semi_march<G, T, 0, false>) : go(k_semi_march<G, T, 1, false>);
}

#define GL_MARCH_INST(G, T) \
  template void launch_semi_march<G, T>(const T*, const T*, const Geom&, const StepConst&, int, const MarchIter&, \
                                        hipStream_t);
GL_MARCH_INST(Su2<double>, double)
GL_MARCH_INST(Su3<double>, double)
GL_MARCH_INST(Su2<float>, float)
GL_MARCH_INST(Su3<float>, float)

}  // namespace gl
