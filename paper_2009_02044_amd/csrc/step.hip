// Leapfrog step with the CPIC charge hop (Sec. 3: eqs. lattice_1, lattice_2,
// plaquette, continuity and the nearest-grid-point transport rule).
//
// One thread owns one site x and its three links (small lattices: one link).  It forms the force terms
//   f_i = sum_{j != i} a_j^-2 P(U_{i,j}(x) + U_{i,-j}(x))
// plaquette by plaquette (stencil.h: plaquette_forces; a forward plaquette serves
// both of its directions), then for each direction updates
//   E_i += dt ( -(1/a_i) f_i + j_i ),   U_i' = exp(i a_i dt E_i) U_i,
// writing U' into the second link buffer (old links stay readable by the
// neighbours) and E in place.  On a hop step the z-link update also moves both
// charge populations one cell with parallel transport and adds the current that
// satisfies the continuity equation exactly:
//   B (+z): rho_B(x+z) <- U_z^dag(x) rho_B(x) U_z(x),     j_z(x) -= (a_L/dt) rho_B(x)
//   A (-z): rho_A(x)   <- U_z(x) rho_A(x+z) U_z^dag(x),   j_z(x) += (a_L/dt) rho_A'(x)
// With co-moving charge storage both rewrites are in place (one slot per thread).
#include <type_traits>
#include "internal.h"
#include "stencil.h"
#include "reduce.h"

namespace gl {

template <typename R> __device__ __forceinline__ M3<double> to_double(const M3<R>& a) {
  M3<double> r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) { r.re[i][j] = (double)a.re[i][j]; r.im[i][j] = (double)a.im[i][j]; }
  return r;
}
template <typename R> __device__ __forceinline__ Q2<double> to_double(const Q2<R>& a) {
  Q2<double> r;
#pragma unroll
  for (int k = 0; k < 4; ++k) r.q[k] = (double)a.q[k];
  return r;
}

// Work-group size of the step kernel.
constexpr int LF_BS = 256;

// Observables gathered by an observing step (FP64): the E and B parts of T^{mu nu} at the
// integer time of the state the step starts from (E averaged over the two half steps,
// B from the forward plaquettes) and a non-finite flag (the Gauss-residual pass before the
// step measures the link unitarity).  The
// plaquette sums hand it each forward plaquette (plane<K>); the S_L terms are formed
// there, with E_i(t + dt/2) computed as the link update computes it, so that no
// projection stays live until the link update.
template <typename G, typename T> struct ObsAcc {
  static constexpr bool UNITARY = false;   // links as stored
  double EL2 = 0.0, ET2 = 0.0, sl = 0.0;
  bool bad = false;
  const T* E;
  uint32_t s;
  int64_t Vp;
  StepConst c;
  double inv_a2[3];
  double* trs;
  // S_L = sum_a (Ebar_x^a P(U_xz)^a / (a_z a_x) + Ebar_y^a P(U_yz)^a / (a_y a_z)).  The real
  // traces of the forward plaquettes (for B^2) are parked in the work-group's LDS,
  // trs[K LF_BS + t], until the end of the step: carried in registers they would hold the
  // step at one wave per SIMD.
  template <int K>
  __device__ __forceinline__ void plane(const typename G::Alg& p, typename G::Real tr, const typename G::Alg& fi) {
    trs[K * LF_BS + threadIdx.x] = (double)tr;
    if constexpr (K > 0) {
      constexpr int i = K - 1;
      typename G::Alg eo;
      load_alg_own(eo, E, i, s, Vp);
      const double ai = c.a[i];
      const T kf = (T)(-c.dt / ai);
      double d = 0.0;
#pragma unroll
      for (int k = 0; k < G::NG; ++k) {
        const T en = fmx(kf, fi.c[k], eo.c[k]);
        d += 0.5 * ((double)eo.c[k] + (double)en) * (double)p.c[k];
      }
      sl += d / (c.a[2] * ai);
      // SU(3): summed here, otherwise the products of this plane wait at the end of the step, with its
      // links in registers (38 spilled; 512 x 64 x 64 814 -> 651 us).  SU(2) spills nothing without:
      // 256 x 128 x 128 608 us with, 587 us without.
      if constexpr (G::NC == 3) asm volatile("" : "+v"(sl));
    }
  }
};

// Update of link (x, i) from the force term f_i of plaquette_forces (F_i = -f_i / a_i);
// the z-link thread also hops the charges.
// FROM: the E and the charges of the state before are read from elsewhere (a step in place adds
// no offsets: read through a second base, the SU(2) FP64 kernel holds 4 registers more and a wave
// per SIMD less, 512 x 64 x 64 2.73 -> 2.80 ms for 16 steps).
template <typename G, typename T, bool HOP, bool OBS = false, bool FROM = false>
__device__ __forceinline__ void finish_link(const typename G::Link& Ui, const typename G::Alg& fi,
                                            T* __restrict__ Unew, T* __restrict__ E, T* __restrict__ rhoA,
                                            T* __restrict__ rhoB, const Geom& g, const StepConst& c, Site x,
                                            uint32_t s, int i, bool reunit, ObsAcc<G, T>* oa = nullptr,
                                            StepFrom from = {}) {
  using L = typename G::Link;
  using A = typename G::Alg;
  constexpr int NG = G::NG;
  const int64_t Vp = g.Vp;
  // i is a run-time value: select the spacing (no indexed local array)
  const double ai = i == 0 ? c.a[0] : (i == 1 ? c.a[1] : c.a[2]);
  A e;
  load_alg_own(e, FROM ? E + from.E : E, i, s, Vp);
  A eo;
  if constexpr (OBS) eo = e;
  const T kf = (T)(-c.dt / ai);
#pragma unroll
  for (int k = 0; k < NG; ++k) e.c[k] = fmx(kf, fi.c[k], e.c[k]);
  if (HOP && c.hop && i == 2) {
    const uint32_t sB = site_index(g, x.x, x.y, slotB(x.z, c.offB, g.nz));
    const uint32_t sA = site_index(g, x.x, x.y, slotA(wrap_add(x.z, 1, g.nz), c.offA, g.nz));
    A rb, ra;
    load_alg_own(rb, FROM ? rhoB + from.rho : rhoB, 0, sB, Vp);
    load_alg_own(ra, FROM ? rhoA + from.rho : rhoA, 0, sA, Vp);
    A rbn = G::transport(Ui, rb);
    A ran = G::transport_inv(Ui, ra);
    store_alg(rbn, rhoB, 0, sB, Vp);
    store_alg(ran, rhoA, 0, sA, Vp);
    // dt * j_z = a_L (rho_A' - rho_B)
    const T al = (T)c.a[2];
#pragma unroll
    for (int k = 0; k < NG; ++k) e.c[k] += al * (ran.c[k] - rb.c[k]);
  }
  store_alg(e, E, i, s, Vp);
  if constexpr (OBS) {
    // E^2 averaged over the half steps
    const double e2 = 0.5 * (norm2(eo) + norm2(e));
    if (i == 2) oa->EL2 = e2; else oa->ET2 += e2;
#pragma unroll
    for (int k = 0; k < NG; ++k) oa->bad |= !isfinite((double)e.c[k]);
  }
  L Un = G::template expi_mul<true>(e, (T)(ai * c.dt), Ui);
  if (reunit) {
    // projection back onto SU(N) in double arithmetic
    using Gd = typename GroupOf<G::NC, double>::type;
    store_link(Gd::reunit(to_double(Un)), Unew, i, s, Vp);
  } else {
    store_link(Un, Unew, i, s, Vp);
  }
}

// The whole site update from plaquette forces.
template <typename G, typename T, bool HOP, bool XS, int OWN, bool OBS = false, bool FROM = false>
__device__ __forceinline__ void update_site(const T* __restrict__ U, T* __restrict__ Unew, T* __restrict__ E,
                                            T* __restrict__ rhoA, T* __restrict__ rhoB, const Geom& g,
                                            const StepConst& c, const double* inv_a2, Site x, uint32_t s,
                                            bool reunit, typename Vec16<T>::type* slot, uint32_t TB,
                                            ObsAcc<G, T>* oa = nullptr, StepFrom from = {}) {
  using L = typename G::Link;
  const GlobalLinks<T> fetch{U, g.Vp};
  const OwnLinks<G, T, OWN> own(fetch, s, slot, threadIdx.x, TB);
  typename G::Alg f[3];
  if constexpr (OBS) plaquette_forces<G, XS, true>(fetch, own, g, x, inv_a2, f, oa);
  else plaquette_forces<G, XS>(fetch, own, g, x, inv_a2, f);
#pragma unroll 1
  for (int i = 0; i < 3; ++i) {
    L Ui;
    own(Ui, i);
    typename G::Alg fi;
#pragma unroll
    for (int k = 0; k < G::NG; ++k) fi.c[k] = i == 0 ? f[0].c[k] : (i == 1 ? f[1].c[k] : f[2].c[k]);
    finish_link<G, T, HOP, OBS, FROM>(Ui, fi, Unew, E, rhoA, rhoB, g, c, x, s, i, reunit, oa, from);
  }
}

#ifndef GL_OWN64
#define GL_OWN64 OWN_LDS
#endif
#ifndef GL_OWN32
#define GL_OWN32 OWN_LDS
#endif
template <typename G, typename T> struct OwnMode {
  static constexpr int value = sizeof(T) == 8 ? GL_OWN64 : GL_OWN32;
};
// LDS for the own-link slots of a work-group of TB threads (one element when unused)
template <typename G, typename T, int TB> struct OwnLds {
  static constexpr int N = OwnMode<G, T>::value == OWN_LDS ? 3 * OwnSlot<G, T>::NCH * TB : 1;
};

#ifndef GL_LF_WAVES
#define GL_LF_WAVES 1
#endif
// One thread per site, the three directions in turn.  OBS: also gather the observables of the state the step starts from into the partial
// sums of this work-group (full work-groups only: every thread reaches the reduction).
// The observing variant is held to two waves per SIMD (its traces live in LDS, below).
// RU: the step also reunitarises the new links (in double arithmetic, before the store).
template <typename G, typename T, bool HOP, bool XS, bool OBS = false, bool RU = false, bool FROM = false>
__global__ void __launch_bounds__(LF_BS, OBS ? 2 : GL_LF_WAVES) k_leapfrog(const T* __restrict__ U, T* __restrict__ Unew,
                                                                 T* __restrict__ E, T* __restrict__ rhoA,
                                                                 T* __restrict__ rhoB, Geom g, StepConst c,
                                                                 ColMap m, double* __restrict__ partial,
                                                                 StepFrom from) {
  Site x;
  uint32_t s;
  __shared__ typename Vec16<T>::type slot[OwnLds<G, T, LF_BS>::N];
  if (!col_map_site(g, m, blockIdx.x, threadIdx.x, LF_BS, x, s)) return;
  const double inv_a2[3] = {1.0 / (c.a[0] * c.a[0]), 1.0 / (c.a[1] * c.a[1]), 1.0 / (c.a[2] * c.a[2])};
  if constexpr (!OBS) {
    update_site<G, T, HOP, XS, OwnMode<G, T>::value, false, FROM>(U, Unew, E, rhoA, rhoB, g, c, inv_a2, x, s, RU, slot,
                                                                  LF_BS, nullptr, from);
  } else {
    __shared__ double trs[3 * LF_BS];
    ObsAcc<G, T> oa;
    oa.trs = trs;
    oa.E = E;
    oa.s = s;
    oa.Vp = g.Vp;
    oa.c = c;
#pragma unroll
    for (int k = 0; k < 3; ++k) oa.inv_a2[k] = inv_a2[k];
    update_site<G, T, HOP, XS, OwnMode<G, T>::value, true>(U, Unew, E, rhoA, rhoB, g, c, inv_a2, x, s, false, slot,
                                                           LF_BS, &oa);
    // B^2 = 4/(a_i a_j)^2 Re Tr(1 - U_ij) (U_{z,x} = U_{x,z}^dag has the same trace); each
    // thread reads back only its own trace slots
    const double nc = (double)G::NC;
    const double BL2 = 4.0 * inv_a2[0] * inv_a2[1] * (nc - trs[threadIdx.x]);
    double BT2 = 4.0 * inv_a2[0] * inv_a2[2] * (nc - trs[LF_BS + threadIdx.x]);
    BT2 += 4.0 * inv_a2[1] * inv_a2[2] * (nc - trs[2 * LF_BS + threadIdx.x]);
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    acc[Q_EPS] = 0.5 * (oa.EL2 + oa.ET2 + BL2 + BT2);
    acc[Q_PL] = 0.5 * (oa.ET2 + BT2 - oa.EL2 - BL2);
    acc[Q_PT] = 0.5 * (oa.EL2 + BL2);
    acc[Q_SL] = oa.sl;
    acc[Q_BAD] = (oa.bad || !isfinite(acc[Q_EPS])) ? 1.0 : 0.0;
    int zb;
    uint32_t slot;
    col_map_block(m, blockIdx.x, zb, slot);
    const unsigned mask = (1u << Q_EPS) | (1u << Q_PL) | (1u << Q_PT) | (1u << Q_SL) | (1u << Q_BAD);
    block_reduce_write<LF_BS, 1u << Q_BAD>(acc, mask, partial + ((int64_t)x.z * col_map_slots_per_layer(m) + slot) * NQ);
  }
}

// One thread per link (blockIdx.y: direction), for lattices that leave most of the chip idle
// with a thread per site: the serial work of a thread, which decides there, is 0.4 of the
// site's.  Each link's force comes out of the same operations in the same order as the site
// kernel's, so the state does not depend on which of the two runs (bitwise).
constexpr int LF_LINK_BS = 64;
template <typename G, typename T, bool HOP, bool XS, bool RU, bool FROM, int D>
__device__ __forceinline__ void update_link(const T* __restrict__ U, T* __restrict__ Unew, T* __restrict__ E,
                                            T* __restrict__ rhoA, T* __restrict__ rhoB, const Geom& g,
                                            const StepConst& c, const double* inv_a2, Site x, uint32_t s,
                                            StepFrom from) {
  const GlobalLinks<T> fetch{U, g.Vp};
  const OwnLinks<G, T, OWN_REGS> own(fetch, s, nullptr, 0, 0);
  typename G::Alg f[3];
  plaquette_forces<G, XS, false, 1 << D>(fetch, own, g, x, inv_a2, f);
  finish_link<G, T, HOP, false, FROM>(own.O[D], f[D], Unew, E, rhoA, rhoB, g, c, x, s, D, RU, nullptr, from);
}
template <typename G, typename T, bool HOP, bool XS, bool RU, bool FROM>
__global__ void __launch_bounds__(LF_LINK_BS) k_leapfrog_link(const T* __restrict__ U, T* __restrict__ Unew,
                                                              T* __restrict__ E, T* __restrict__ rhoA,
                                                              T* __restrict__ rhoB, Geom g, StepConst c, ColMap m,
                                                              StepFrom from) {
  Site x;
  uint32_t s;
  if (!col_map_site(g, m, blockIdx.x, threadIdx.x, LF_LINK_BS, x, s)) return;
  const double inv_a2[3] = {1.0 / (c.a[0] * c.a[0]), 1.0 / (c.a[1] * c.a[1]), 1.0 / (c.a[2] * c.a[2])};
  if (blockIdx.y == 0) update_link<G, T, false, XS, RU, FROM, 0>(U, Unew, E, rhoA, rhoB, g, c, inv_a2, x, s, from);
  else if (blockIdx.y == 1) update_link<G, T, false, XS, RU, FROM, 1>(U, Unew, E, rhoA, rhoB, g, c, inv_a2, x, s, from);
  else update_link<G, T, HOP, XS, RU, FROM, 2>(U, Unew, E, rhoA, rhoB, g, c, inv_a2, x, s, from);
}

// Whether a step takes a thread per link.  Both kernels take as long as the XCD with the most layers,
// so the rule counts there: the waves of the link kernel, and for SU(3) FP64 the work-groups of the
// site kernel, which runs one per CU as long as there are 32 of them (0.30 ms for 16 steps) and a second
// one beside it above (0.51 - 0.64 ms); its link kernel runs one wave per SIMD (1.0 us more for every
// wave of the XCD).  With rows inside wavefronts (nt = 16, 32, 64) the site kernel is the cheaper for it.
// 16 steps, site against link kernel (us):
//   SU(3) FP64: 252 waves 295 / 277, 324 waves 309 / 366, 384 waves 332 / 391; above 32 work-groups:
//     375 waves 508 / 389, 480 waves 541 / 519, 540 waves 559 / 585
//   SU(2) FP64: 540 waves 165 / 167, 621 waves 190 / 152, 672 waves 198 / 225; rows inside: 576 waves 184 /
//     175, 624 waves 176 / 182
//   SU(3) FP32: 618 waves 334 / 319, 621 waves 399 / 299, 672 waves 342 / 368; inside: 576 waves 314 / 289,
//     624 waves 315 / 330
//   SU(2) FP32: 672 waves 143 / 123, 864 waves 175 / 140; inside: 624 waves 116 / 111, 672 waves 116 / 121
// (64 x 8 x 8, in this order: 219 / 114, 97 / 59, 195 / 102, 87 / 65.)
// Layers of at most 64 sites leave three of a site work-group's four waves without work: 1250 x 8 x 8
// 746 / 533, 150 / 145, 427 / 280, 111 / 95 (measured up to 80 000 sites).
constexpr int64_t LF_LINK_SMALL = 81920;
template <typename G, typename T> bool step_by_links(const Geom& g) {
  if (g.layer <= LF_LINK_BS && g.V <= LF_LINK_SMALL) return true;
  const int64_t waves = 3 * (int64_t)(col_map_blocks(g, col_map(g, LF_LINK_BS)) / NXCD);
  const bool inside = rows_in_wavefronts(g.nt);
  if (G::NC == 3 && sizeof(T) == 8)
    return waves <= (col_map_blocks(g, col_map(g, LF_BS)) / NXCD <= 32 ? 256 : 512);
  if (G::NC == 2 && sizeof(T) == 4) return waves <= (inside ? 640 : 864);
  return waves <= (inside ? 600 : 640);
}

// Sites of a layer up to which it is swept whole: half of what the work-groups in flight on an XCD
// cover (32 CUs, 4 SIMDs, 64 sites a wave), which is 2, 4, 4 and 8 waves per SIMD for SU(3) FP64,
// SU(3) FP32, SU(2) FP64 and SU(2) FP32.  16 steps, whole against bands: SU(3) FP64 64 x 97 x 97 3169 /
// 3042 us, 128 x 128 x 128 10116 / 9646; SU(3) FP32 32 x 128 x 128 1289 / 1311, 128 x 150 x 150 7051 /
// 6893; SU(2) FP64 64 x 100 x 100 1027 / 1047, 32 x 128 x 128 853 / 867, 128 x 150 x 150 4730 / 4552; SU(2)
// FP32 128 x 150 x 150 2441 / 2481, 40 x 192 x 192 990 / 896.
template <typename G, typename T>
constexpr int64_t WHOLE_LAYER = sizeof(T) == 8 ? (G::NC == 3 ? 9216 : 16384) : (G::NC == 3 ? 16384 : 32768);

template <typename G, typename T>
void launch_leapfrog(const T* U, T* Unew, T* E, T* rhoA, T* rhoB, const Geom& g, const StepConst& c,
                     bool reunit, hipStream_t st, StepFrom from) {
  // rows inside wavefronts: x neighbours from other lanes
  const bool xs = rows_in_wavefronts(g.nt);
  const bool link = step_by_links<G, T>(g);
  const int bs = link ? LF_LINK_BS : LF_BS;
  const ColMap m = col_map(g, bs, WHOLE_LAYER<G, T>);
  const dim3 grid(col_map_blocks(g, m), link ? 3 : 1);
  auto pick = [&](auto hop, auto xn, auto ru, auto fr) {
    constexpr bool H = decltype(hop)::value, X = decltype(xn)::value, R = decltype(ru)::value,
                   F = decltype(fr)::value;
    if (link)
      hipLaunchKernelGGL((k_leapfrog_link<G, T, H, X, R, F>), grid, dim3(bs), 0, st, U, Unew, E, rhoA, rhoB, g, c, m,
                         from);
    else
      hipLaunchKernelGGL((k_leapfrog<G, T, H, X, false, R, F>), grid, dim3(bs), 0, st, U, Unew, E, rhoA, rhoB, g, c,
                         m, nullptr, from);
  };
  using Y = std::true_type;
  using N = std::false_type;
  auto with = [&](auto fr) {
    if (!reunit) {
      if (c.hop) xs ? pick(Y{}, Y{}, N{}, fr) : pick(Y{}, N{}, N{}, fr);
      else xs ? pick(N{}, Y{}, N{}, fr) : pick(N{}, N{}, N{}, fr);
    } else {
      if (c.hop) xs ? pick(Y{}, Y{}, Y{}, fr) : pick(Y{}, N{}, Y{}, fr);
      else xs ? pick(N{}, Y{}, Y{}, fr) : pick(N{}, N{}, Y{}, fr);
    }
  };
  if (from.E == 0 && from.rho == 0) with(N{});
  else with(Y{});
}

// The observing step: the leapfrog step that also writes the energy slots of the
// observables of the state it starts from (FP64; nt a multiple of 64, so the column map
// has only full work-groups).  x neighbours come from adjacent lanes when a row lies in a
// wavefront (nt = 64), else from memory, as in the plain step.
template <typename G, typename T>
void launch_leapfrog_observe(const T* U, T* Unew, T* E, T* rhoA, T* rhoB, const Geom& g, const StepConst& c,
                             double* partial, hipStream_t st) {
  const int bs = LF_BS;
  const ColMap m = col_map(g, bs, WHOLE_LAYER<G, T>);
  const unsigned nbc = col_map_blocks(g, m);
  const bool xs = rows_in_wavefronts(g.nt);
  if (c.hop) {
    if (xs) hipLaunchKernelGGL((k_leapfrog<G, T, true, true, true>), dim3(nbc), dim3(bs), 0, st, U, Unew, E, rhoA,
                               rhoB, g, c, m, partial, StepFrom{});
    else hipLaunchKernelGGL((k_leapfrog<G, T, true, false, true>), dim3(nbc), dim3(bs), 0, st, U, Unew, E, rhoA,
                            rhoB, g, c, m, partial, StepFrom{});
  } else {
    if (xs) hipLaunchKernelGGL((k_leapfrog<G, T, false, true, true>), dim3(nbc), dim3(bs), 0, st, U, Unew, E, rhoA,
                               rhoB, g, c, m, partial, StepFrom{});
    else hipLaunchKernelGGL((k_leapfrog<G, T, false, false, true>), dim3(nbc), dim3(bs), 0, st, U, Unew, E, rhoA,
                            rhoB, g, c, m, partial, StepFrom{});
  }
}
template void launch_leapfrog_observe<Su3<double>, double>(const double*, double*, double*, double*, double*,
                                                          const Geom&, const StepConst&, double*, hipStream_t);
template void launch_leapfrog_observe<Su2<double>, double>(const double*, double*, double*, double*, double*,
                                                          const Geom&, const StepConst&, double*, hipStream_t);

// ---- batched form: many events of different sizes in one launch --------------

// Work item = `bs` consecutive sites of one event: one work-group per item, or persistent
// work-groups that loop over the items.  The step number comes
// from device memory so that a captured graph of several steps replays correctly:
// parity of the link buffers, hop flag and charge offsets all follow from it.
GL_HD int64_t hop_count_dev(int64_t s, int64_t p, int64_t q) { return ((2 * s + 1) * p + q) / (2 * q); }

// Per-step values of the batch, from the device step counter.
struct BatchStep {
  int64_t st, S0;
  bool hop, reunit;
  double inv_a2[3];
};
__device__ __forceinline__ BatchStep batch_step_of(const BatchConst& bc, const int64_t* __restrict__ ctr) {
  BatchStep b;
  b.st = ctr[0];
  const int64_t S1 = hop_count_dev(b.st, bc.hop_p, bc.hop_q);
  b.S0 = hop_count_dev(b.st - 1, bc.hop_p, bc.hop_q);
  b.hop = S1 > b.S0;
  b.reunit = bc.reunit_every > 0 && ((b.st + 1) % bc.reunit_every) == 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) b.inv_a2[k] = 1.0 / (bc.a[k] * bc.a[k]);
  return b;
}

// One work item: blockDim.x consecutive sites of one event.
template <typename G, typename T>
__device__ __forceinline__ void batch_item(char* __restrict__ pool, const EventDesc* __restrict__ ev,
                                           const uint32_t* __restrict__ item_event, const BatchConst& bc,
                                           const BatchStep& b, uint32_t item, typename Vec16<T>::type* slot) {
  const EventDesc d = ev[item_event[item]];
  const uint32_t s = (item - d.item0) * blockDim.x + threadIdx.x;
  if (s >= (uint32_t)d.g.V) return;
  StepConst c;
  c.a[0] = bc.a[0]; c.a[1] = bc.a[1]; c.a[2] = bc.a[2];
  c.dt = bc.dt;
  c.hop = b.hop ? 1 : 0;
  const int64_t off = (d.off0 + (b.S0 - d.hops0)) % d.g.nz;
  c.offA = (int)off;
  c.offB = (int)off;
  c.scheme = 0;
  const bool odd = (b.st & 1) != 0;
  const T* U = (const T*)(pool + (odd ? d.Uodd : d.Ueven));
  T* Un = (T*)(pool + (odd ? d.Ueven : d.Uodd));
  Site x;
  x.x = (int)(s % (uint32_t)d.g.nt);
  x.y = (int)((s / (uint32_t)d.g.nt) % (uint32_t)d.g.nt);
  x.z = (int)(s / (uint32_t)d.g.layer);
  // item = 64-aligned sites of one event: rows lie in wavefronts when nt divides 64
  constexpr int K = OwnMode<G, T>::value;
  T *E = (T*)(pool + d.E), *rA = (T*)(pool + d.rhoA), *rB = (T*)(pool + d.rhoB);
  const uint32_t TB = blockDim.x;
  const Geom g = d.g;
  // the hop branch inside is uniform over the launch (HOP = true only enables it)
  if (rows_in_wavefronts(g.nt))
    update_site<G, T, true, true, K>(U, Un, E, rA, rB, g, c, b.inv_a2, x, s, b.reunit, slot, TB);
  else
    update_site<G, T, true, false, K>(U, Un, E, rA, rB, g, c, b.inv_a2, x, s, b.reunit, slot, TB);
}

// Items are dealt to the XCDs in chunks of 64 (xcd_chunk_remap): 2.5% faster than one by one
// on a mix of 64 events, which keeps the XCDs' shares of the events balanced.
constexpr uint32_t BATCH_XCD_CHUNK = 64;

// Persistent form: `grid` work-groups loop over the items (a grid that is a multiple of 8
// keeps each work-group's indices on its own XCD).
template <typename G, typename T>
__global__ void __launch_bounds__(256) k_batch_step(char* __restrict__ pool, const EventDesc* __restrict__ ev,
                                                    const uint32_t* __restrict__ item_event, BatchConst bc,
                                                    const int64_t* __restrict__ ctr) {
  const BatchStep b = batch_step_of(bc, ctr);
  __shared__ typename Vec16<T>::type slot[OwnLds<G, T, 256>::N];
  for (uint32_t v = blockIdx.x; v < bc.items; v += gridDim.x)
    batch_item<G, T>(pool, ev, item_event, bc, b, xcd_chunk_remap<BATCH_XCD_CHUNK>(v, bc.items), slot);
}

// One work-group per item.  Without the loop the FP32 kernel fits 128 registers and runs at
// four waves per SIMD (the loop costs it ~23 registers and a wave).
template <typename G, typename T>
__global__ void __launch_bounds__(256, sizeof(T) == 4 ? 4 : 1)
    k_batch_step_flat(char* __restrict__ pool, const EventDesc* __restrict__ ev,
                      const uint32_t* __restrict__ item_event, BatchConst bc, const int64_t* __restrict__ ctr) {
  const BatchStep b = batch_step_of(bc, ctr);
  __shared__ typename Vec16<T>::type slot[OwnLds<G, T, 256>::N];
  if (blockIdx.x < bc.items)
    batch_item<G, T>(pool, ev, item_event, bc, b, xcd_chunk_remap<BATCH_XCD_CHUNK>(blockIdx.x, bc.items), slot);
}

// advance the device step counter (one lane writes)
__global__ void k_batch_tick(int64_t* ctr) {
  if (threadIdx.x == 0) {
    const int64_t v = ctr[0];
    ctr[threadIdx.x] = v + 1;
  }
}

template <typename G, typename T>
void launch_batch_step(char* pool, const EventDesc* ev, const uint32_t* item_event, const BatchConst& bc,
                       const int64_t* ctr, int grid, int bs, hipStream_t st) {
  if (grid > 0)
    hipLaunchKernelGGL((k_batch_step<G, T>), dim3((unsigned)grid), dim3((unsigned)bs), 0, st, pool, ev, item_event, bc,
                       ctr);
  else
    hipLaunchKernelGGL((k_batch_step_flat<G, T>), dim3(bc.items), dim3((unsigned)bs), 0, st, pool, ev, item_event,
                       bc, ctr);
}
void launch_batch_tick(int64_t* ctr, hipStream_t st) { hipLaunchKernelGGL(k_batch_tick, dim3(1), dim3(64), 0, st, ctr); }

template void launch_batch_step<Su2<double>, double>(char*, const EventDesc*, const uint32_t*, const BatchConst&, const int64_t*, int, int, hipStream_t);
template void launch_batch_step<Su3<double>, double>(char*, const EventDesc*, const uint32_t*, const BatchConst&, const int64_t*, int, int, hipStream_t);
template void launch_batch_step<Su2<float>, float>(char*, const EventDesc*, const uint32_t*, const BatchConst&, const int64_t*, int, int, hipStream_t);
template void launch_batch_step<Su3<float>, float>(char*, const EventDesc*, const uint32_t*, const BatchConst&, const int64_t*, int, int, hipStream_t);

template void launch_leapfrog<Su2<double>, double>(const double*, double*, double*, double*, double*, const Geom&, const StepConst&, bool, hipStream_t, StepFrom);
template void launch_leapfrog<Su3<double>, double>(const double*, double*, double*, double*, double*, const Geom&, const StepConst&, bool, hipStream_t, StepFrom);
template void launch_leapfrog<Su2<float>, float>(const float*, float*, float*, float*, float*, const Geom&, const StepConst&, bool, hipStream_t, StepFrom);
template void launch_leapfrog<Su3<float>, float>(const float*, float*, float*, float*, float*, const Geom&, const StepConst&, bool, hipStream_t, StepFrom);

}  // namespace gl
