// Initial conditions of two MV nuclei with finite longitudinal extent, computed on
// the GPU in double precision (Sec. 2: Gaussian W[rho] and the Fourier solution of
// the transverse Poisson equation with IR regulator m and UV cutoff Lambda;
// Sec. 3: eqs. single_sheet, 3d_colorfield_1, 3d_colorfield_2, the temporal gauge,
// and the CPIC charges that satisfy eq. gauss).
//
// 1. phi^a_N = DFT^-1[ rho~^a_N Theta(Lambda - |k~|) / (k~^2 + m^2) ] on the nt x nt
//    transverse torus, k~^2 = (2/a_T)^2 (sin^2(pi kx/nt) + sin^2(pi ky/nt)), by four
//    separable direct DFT passes (nt <= a few hundred, one-shot per event; k_dft).
// 2. Wilson lines V_N(x, t) = exp(-i Lambda_N(z, t) phi_N(x_T)): the colour structure
//    of a single sheet does not depend on z, so the path ordering is trivial and the
//    cumulative normalised Gaussian profile is
//      Lambda_B = erfc((z - z_B - (t - t0)) / (sqrt 2 sigma)) / 2   (B moves +z),
//      Lambda_A = erfc(-(z - z_A + (t - t0)) / (sqrt 2 sigma)) / 2  (A moves -z).
//    With ns sheets (colour structure varying along the beam axis, independent
//    charges per piece of equal profile weight, Sec. 3 after eq. single_sheet and
//    Sec. 5) the line is the path-ordered product
//      V_N = exp(-i lambda_0 phi_{N,0}) ... exp(-i lambda_{ns-1} phi_{N,ns-1}),
//      lambda_k = clamp(ns Lambda_N - k, 0, 1),
//    the sheet crossed later on the right (V^dag, the path-ordered exponential of
//    Sec. 2, has later points on the left); with A_i = V d_i V^dag / (ig) the field
//    strength inside piece k is then sheet k's own, rotated by the completed pieces
//    (gauge covariance); sheets not reached yet (lambda_k = 0) are 1.
// 3. U_i = [V_A(x) V_A^dag(x+i)] [V_B(x) V_B^dag(x+i)] (i = x, y), U_z = 1 except the
//    periodic seam U_z(x_T, nz-1) = V_A(x_T, nz-1) V_B^dag(x_T, 0), at t0 and t0 - dt.
// 4. E_i(t0 - dt/2) = -i Log(U_i(t0) U_i^dag(t0 - dt)) / (a_i dt), principal Log.
// 5. rho = sum_i [E_i(x) - U_i^dag(x-i) E_i(x-i) U_i(x-i)] / a_i at U(t0); layers
//    z < nz/2 go to nucleus B, the others to nucleus A.
#include <algorithm>
#include <type_traits>
#include "internal.h"

namespace gl {

size_t ic_work_doubles(const Geom& g, int ng) { return (size_t)6 * 2 * ng * g.layer; }

// The four DFT passes of nb real nt x nt planes.  A real plane's transform at -k is the
// conjugate of that at k, so only kx = 0 .. nt/2 are formed and kept (rows of h = nt/2 + 1
// complex numbers):
//   0: real, forward along x          out[b][y][kx] = sum_u in[b][y][u] e^{-2 pi i kx u / nt}
//   1: forward along y, times 1 / (k~^2 + m^2) and the cut
//   2: inverse along y
//   3: inverse along x, the kx > 0 terms counted twice (not kx = nt/2 of an even nt), / nt^2
// Outputs o and nt - o of a line have conjugate phases, so one thread forms both from the
// sums A = sum x c, B = sum y s, C = sum x s, D = sum y c over the data x + iy and phases c + is:
// half the products.  A work-group takes DFT_LINES lines (rows or columns) of a plane, staged
// in LDS in chunks of DFT_CHUNK terms; the phases e^{2 pi i k / nt} come from a table of nt
// entries in LDS (term u of output o takes entry (o u) mod nt, kept by adding o), so a term
// costs five LDS reads for four lines and two outputs, which is what bounds a pass, and no
// global latency.  Before, every term evaluated its own sincospi, read its datum from memory
// and all nt columns were formed: 284 us a pass on 16 planes of 192 x 192 (18-20 us on
// 64 x 64), now 14-30 us (5-11 us).  The table alone, without staging, took 45-76 us: each
// term waited for its load.
// Sums are formed in blocks of DFT_BLOCK terms: a rounding then weighs a block's sum, not the whole
// line's.  With half a spectrum the errors of +-k no longer cancel, and plain sums have phi 2-5% further
// off than the full transform (9.0e-16 against 8.6e-16 of phi at nt = 192); in blocks 4.1e-16.
constexpr int DFT_BS = 256, DFT_LINES = 4, DFT_CHUNK = 256, DFT_FETCH = 8, DFT_BLOCK = 16;
constexpr int DFT_TABLE_MAX = 2048;   // 32 KB of LDS; longer lines evaluate each phase
struct DftConst {
  int nt, h, nb;
  double a_T, m_ir, uv_cut;
};
__device__ __forceinline__ double2 dft_phase(int k, int nt) {
  double2 w;
  sincospi(2.0 * (double)k / nt, &w.y, &w.x);
  return w;
}
// sin(pi k / nt) and sin(pi (nt - k) / nt), each as rounded
struct DftSine {
  double p, m;
};
__device__ __forceinline__ DftSine dft_sine(int k, const DftConst& c) {
  return DftSine{sinpi((double)k / c.nt), sinpi((double)(k ? c.nt - k : 0) / c.nt)};
}
// The weight of a mode (kx, ky) of the half spectrum, and with neg of (kx, -ky): the mean over k and -k of
// 1 / (k~^2 + m^2) Theta(Lambda - |k~|).  The two sines round differently, so a cut at a mode's |k~| can
// fall between them; the real part of the transform then holds half of the mode, along x as along y.
__device__ __forceinline__ double dft_weight(const DftSine& x, const DftSine& y, bool neg, const DftConst& c) {
  const double yp = neg ? y.m : y.p, ym = neg ? y.p : y.m, a2 = (2.0 / c.a_T) * (2.0 / c.a_T);
  const double kp = a2 * (yp * yp + x.p * x.p);
  double w = 1.0;
  if (c.uv_cut > 0.0) {
    const double km = a2 * (ym * ym + x.m * x.m);
    w = (sqrt(kp) > c.uv_cut ? 0.0 : 0.5) + (sqrt(km) > c.uv_cut ? 0.0 : 0.5);
  }
  return w / (kp + c.m_ir * c.m_ir);
}
// terms 0 .. n - 1 in blocks of B, done() after each
template <int B, int UNROLL, typename F, typename D>
__device__ __forceinline__ void in_blocks(int n, F&& term, D&& done) {
  int u = 0;
  for (; u + B <= n; u += B) {
#pragma unroll UNROLL
    for (int f = 0; f < B; ++f) term(u + f);
    done();
  }
  if (u == n) return;
  for (; u < n; ++u) term(u);
  done();
}
// (held to few waves per SIMD: with registers for more, the compiler waits for every LDS read)
template <int MODE, bool TABLE>
__global__ void __launch_bounds__(DFT_BS) __attribute__((amdgpu_waves_per_eu(1, 2)))
k_dft(const double* __restrict__ in, double* __restrict__ out, DftConst c) {
  constexpr bool ROWS = MODE == 0 || MODE == 3;         // lines are rows, else columns
  constexpr int W = MODE == 0 ? 1 : 2;                  // doubles per datum
  extern __shared__ double2 tab[];
  __shared__ double2 buf[DFT_CHUNK * DFT_LINES * W / 2];
  double* bd = (double*)buf;                            // [term][line][W]
  const int nt = c.nt, h = c.h, b = blockIdx.z;
  const int len = MODE == 3 ? h : nt;                   // terms of a sum
  const int nline = ROWS ? nt : h;
  const int l0 = blockIdx.x * DFT_LINES;
  const int o = blockIdx.y * DFT_BS + threadIdx.x;      // this output and nt - o
  if constexpr (TABLE)
    for (int k = threadIdx.x; k < nt; k += blockDim.x) tab[k] = dft_phase(k, nt);
  double sa[DFT_LINES], sb[DFT_LINES], sc[DFT_LINES], sd[DFT_LINES];
#pragma unroll
  for (int r = 0; r < DFT_LINES; ++r) sa[r] = sb[r] = sc[r] = sd[r] = 0.0;
  const int step = o < h ? o : 0;
  int k = 0;
  for (int u0 = 0; u0 < len; u0 += DFT_CHUNK) {
    const int n = min(DFT_CHUNK, len - u0);
    __syncthreads();
    // DFT_FETCH loads in flight per thread
    for (int q0 = threadIdx.x; q0 < n * DFT_LINES; q0 += DFT_FETCH * blockDim.x) {
      double2 v[DFT_FETCH];
#pragma unroll
      for (int f = 0; f < DFT_FETCH; ++f) {
        const int q = min(q0 + f * (int)blockDim.x, n * DFT_LINES - 1);
        const int r = ROWS ? q / n : q % DFT_LINES, u = ROWS ? q % n : q / DFT_LINES;
        const int l = min(l0 + r, nline - 1);           // lines past the end repeat the last one
        const int64_t at = ROWS ? ((int64_t)b * nt + l) * len + u0 + u : ((int64_t)b * nt + u0 + u) * h + l;
        if constexpr (W == 1) v[f].x = in[at];
        else v[f] = ((const double2*)in)[at];
      }
#pragma unroll
      for (int f = 0; f < DFT_FETCH; ++f) {
        const int q = min(q0 + f * (int)blockDim.x, n * DFT_LINES - 1);
        const int r = ROWS ? q / n : q % DFT_LINES, u = ROWS ? q % n : q / DFT_LINES;
        // pass 3: the terms kx > 0 stand for -kx too (not kx = nt/2 of an even nt)
        const double m = MODE == 3 && u0 + u != 0 && 2 * (u0 + u) != nt ? 2.0 : 1.0;
        if constexpr (W == 1) bd[u * DFT_LINES + r] = v[f].x;
        else buf[u * DFT_LINES + r] = make_double2(m * v[f].x, m * v[f].y);
      }
    }
    __syncthreads();
    double pa[DFT_LINES], pb[DFT_LINES], pc[DFT_LINES], pd[DFT_LINES];   // sums of a block
#pragma unroll
    for (int r = 0; r < DFT_LINES; ++r) pa[r] = pb[r] = pc[r] = pd[r] = 0.0;
    in_blocks<DFT_BLOCK, 4>(n, [&](int u) __attribute__((always_inline)) {
      const double2 w = TABLE ? tab[k] : dft_phase(k, nt);
      k += step;
      k = k >= nt ? k - nt : k;
#pragma unroll
      for (int r = 0; r < DFT_LINES; ++r) {
        if constexpr (MODE == 0) {
          const double v = bd[u * DFT_LINES + r];
          pa[r] = fmx(v, w.x, pa[r]);
          pc[r] = fmx(v, w.y, pc[r]);
        } else {
          const double2 v = buf[u * DFT_LINES + r];
          pa[r] = fmx(v.x, w.x, pa[r]);
          pb[r] = fmx(v.y, w.y, pb[r]);
          if constexpr (MODE != 3) {
            pc[r] = fmx(v.x, w.y, pc[r]);
            pd[r] = fmx(v.y, w.x, pd[r]);
          }
        }
      }
    }, [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < DFT_LINES; ++r) {
        sa[r] += pa[r];
        sb[r] += pb[r];
        sc[r] += pc[r];
        sd[r] += pd[r];
        pa[r] = pb[r] = pc[r] = pd[r] = 0.0;
      }
    });
  }
  if (o >= h) return;
  const bool both = MODE != 0 && o != 0 && 2 * o != nt;
  DftSine sy;
  if constexpr (MODE == 1) sy = dft_sine(o, c);
#pragma unroll
  for (int r = 0; r < DFT_LINES; ++r) {
    const int l = l0 + r;
    if (l >= nline) break;
    DftSine sx;
    if constexpr (MODE == 1) sx = dft_sine(l, c);
    auto put = [&](int q, double s) {   // output q, its phases c + s i s
      if constexpr (MODE == 3) {
        out[((int64_t)b * nt + l) * nt + q] = fmx(-s, sb[r], sa[r]) / ((double)nt * nt);
      } else {
        const double f = MODE == 1 ? dft_weight(sx, sy, q != o, c) : 1.0;
        const int64_t at = ROWS ? ((int64_t)b * nt + l) * h + q : ((int64_t)b * nt + q) * h + l;
        ((double2*)out)[at] = make_double2(f * fmx(-s, sb[r], sa[r]), f * fmx(s, sc[r], sd[r]));
      }
    };
    constexpr double fwd = MODE <= 1 ? -1.0 : 1.0;
    put(o, fwd);
    if (both) put(nt - o, -fwd);
  }
}

// The same four passes for small planes in one launch: a work-group holds one plane, its half
// spectrum in LDS between the passes.  Up to 32 x 32, where the separate passes are bound by
// their launches: four passes on 6 planes of 8 x 8 took 16 us, now 5.5 us, on 16 of 32 x 32 42 us, now 16 us; larger planes
// leave too few work-groups busy (one per plane).  Sums in blocks of 4 as above: 3.0e-16 of phi at nt =
// 32, 2.5e-16 at 16 (3.9e-16 and 3.1e-16 with every term its own phase, no half spectrum).
constexpr int DFT_SMALL = 32, DFT_SMALL_BS = 512, DFT_SMALL_BLOCK = 4;
__global__ void __launch_bounds__(DFT_SMALL_BS) k_dft_small(const double* __restrict__ in, double* __restrict__ out,
                                                            DftConst c) {
  __shared__ double2 tab[DFT_SMALL];
  __shared__ double2 f[2][DFT_SMALL * (DFT_SMALL / 2 + 1)];
  __shared__ double g[DFT_SMALL * DFT_SMALL];
  const int nt = c.nt, h = c.h, n2 = nt * nt, t0 = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * n2;
  for (int k = t0; k < nt; k += DFT_SMALL_BS) tab[k] = dft_phase(k, nt);
  for (int k = t0; k < n2; k += DFT_SMALL_BS) g[k] = in[base + k];
  __syncthreads();
  for (int t = t0; t < nt * h; t += DFT_SMALL_BS) {
    const int x = t % h, y = t / h;
    double sr = 0.0, si = 0.0, pr = 0.0, pi = 0.0;
    int k = 0;
    auto done = [&]() { sr += pr; si += pi; pr = pi = 0.0; };
    in_blocks<DFT_SMALL_BLOCK, DFT_SMALL_BLOCK>(nt, [&](int u) {
      const double v = g[y * nt + u];
      const double2 w = tab[k];
      k += x;
      k = k >= nt ? k - nt : k;
      pr = fmx(v, w.x, pr);
      pi = fmx(-v, w.y, pi);
    }, done);
    f[0][t] = make_double2(sr, si);
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 2; ++p) {   // along y: forward with the filter, then inverse
    for (int t = t0; t < nt * h; t += DFT_SMALL_BS) {
      const int x = t % h, y = t / h;
      double sr = 0.0, si = 0.0, pr = 0.0, pi = 0.0;
      int k = 0;
      auto done = [&]() { sr += pr; si += pi; pr = pi = 0.0; };
      in_blocks<DFT_SMALL_BLOCK, DFT_SMALL_BLOCK>(nt, [&](int u) {
        const double2 v = f[p][u * h + x];
        const double2 w = tab[k];
        k += y;
        k = k >= nt ? k - nt : k;
        const double wi = p == 0 ? -w.y : w.y;
        pr += fmx(v.x, w.x, -(v.y * wi));
        pi += fmx(v.x, wi, v.y * w.x);
      }, done);
      const double q = p == 0 ? dft_weight(dft_sine(x, c), dft_sine(y, c), false, c) : 1.0;
      f[1 - p][t] = make_double2(q * sr, q * si);
    }
    __syncthreads();
  }
  for (int t = t0; t < n2; t += DFT_SMALL_BS) {
    const int x = t % nt, y = t / nt;
    double sr = 0.0, pr = 0.0;
    int k = 0;
    auto done = [&]() { sr += pr; pr = 0.0; };
    in_blocks<DFT_SMALL_BLOCK, DFT_SMALL_BLOCK>(h, [&](int u) {
      const double2 v = f[0][y * h + u];
      const double2 w = tab[k];
      k += x;
      k = k >= nt ? k - nt : k;
      const double m = (u == 0 || 2 * u == nt) ? 1.0 : 2.0;
      pr += fmx(m * v.x, w.x, -(m * v.y * w.y));
    }, done);
    out[base + t] = sr / (double)n2;
  }
}

template <typename Gd>
__device__ __forceinline__ typename Gd::Alg sheet_phi(const double* __restrict__ phi, int sheet, int nucleus,
                                                      int64_t t, int64_t layer) {
  typename Gd::Alg p;
  constexpr int NG = Gd::NG;
#pragma unroll
  for (int k = 0; k < NG; ++k) p.c[k] = phi[(((int64_t)sheet * 2 + nucleus) * NG + k) * layer + t];
  return p;
}
// V_N at transverse site t for cumulative profile weight lam of the whole nucleus
template <typename Gd>
__device__ typename Gd::Link wilson(const double* __restrict__ phi, int ns, int nucleus, int64_t t, int64_t layer,
                                    double lam) {
  typename Gd::Link V = Gd::expi(sheet_phi<Gd>(phi, 0, nucleus, t, layer), -fmin(fmax(ns * lam, 0.0), 1.0));
  for (int k = 1; k < ns; ++k) {
    const double lk = fmin(fmax(ns * lam - k, 0.0), 1.0);
    if (lk > 0.0) V = Gd::mul(V, Gd::expi(sheet_phi<Gd>(phi, k, nucleus, t, layer), -lk));
  }
  return V;
}

// distance ahead of the nucleus's centre (A moves -z)
__device__ __forceinline__ double aheadA(double z, double tau, const McvConst& mv) { return -(z - mv.zA + tau); }
__device__ __forceinline__ double aheadB(double z, double tau, const McvConst& mv) { return z - mv.zB - tau; }
__device__ __forceinline__ double profile(double ahead, const McvConst& mv) {
  return 0.5 * erfc(ahead / (1.4142135623730951 * mv.sigma));
}
__device__ __forceinline__ double of_lane(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Links and E of one tile of IC_TX x IC_TY transverse sites at one z per work-group.  A transverse link
// of nucleus N is V_N(x) V_N^dag(x + i), and V_N belongs to a site: each is formed once per tile (and
// once more per neighbouring tile, on the tile's +x and +y rim) and read from LDS by the threads that
// need it, both nuclei at a time, the two times in turn.  SU(3): a thread per link (the first half of the
// work-group x links, the other y links); SU(2): a thread per site.
// Matrices between the exponentials and the stored link are held whole: by two rows, the third
// rebuilt, SU(3) E is 7% (1 sheet) to 19% (8 sheets) further off.  Bound by FP64 arithmetic; with every
// site forming its neighbours' V itself (16 exponentials per site and sheet instead of 4.8) 512 x 64 x 64
// took 0.81 ms and 1.89 ms with 8 sheets, now 0.43 and 0.71 ms (0.40 and 0.64 ms by two rows).
// Layers that the profiles of both times reach equally (the flat parts) take U(t0 - dt) = U(t0).
constexpr int IC_BS = 256, IC_TX = 16, IC_RIM = IC_TX + 1;
template <typename Gd> constexpr int IC_LINKS = Gd::NC == 3 ? 1 : 2;   // of a thread
template <typename Gd> constexpr int IC_TY = IC_BS * IC_LINKS<Gd> / 2 / IC_TX;
template <typename Gd, typename T>
__global__ void __launch_bounds__(IC_BS, 2) k_ic_links(const double* __restrict__ phi, int ns, T* __restrict__ U,
                                                       T* __restrict__ E, Geom g, StepConst c, McvConst mv, int z_first) {
  using L = typename Gd::Link;
  using A = typename Gd::Alg;
  constexpr int NG = Gd::NG, W = FullWidth<L>::value, NL = IC_LINKS<Gd>;
  constexpr int SITES = IC_TX * IC_TY<Gd>, PITCH = IC_RIM * (IC_TY<Gd> + 1);
  __shared__ double v[2 * W * PITCH];   // V_N, real k of tile site p at v[(N W + k) PITCH + p]
  const int x0 = blockIdx.x * IC_TX, y0 = blockIdx.y * IC_TY<Gd>;
  const int i0 = __builtin_amdgcn_readfirstlane(threadIdx.x / SITES);   // first direction (uniform over a wavefront)
  const int tx = threadIdx.x % IC_TX, ty = threadIdx.x % SITES / IC_TX;
  const bool has = x0 + tx < g.nt && y0 + ty < g.nt;
  const uint32_t t = (uint32_t)(min(y0 + ty, g.nt - 1) * g.nt + min(x0 + tx, g.nt - 1));
  const int z = z_first + (int)blockIdx.z;
  if (z == g.nz) {   // the z links of the periodic seam, in work-groups of their own
    if (!has || i0) return;
    const double zs = (g.nz - 1) * c.a[2];
    const uint32_t s = (uint32_t)((g.nz - 1) * g.layer) + t;
    double* park = v + threadIdx.x;   // U(t0), a slot per thread (SITES < PITCH of them)
    L us;
#pragma unroll 1
    for (int q = 0; q < 2; ++q) {
      const double tau = q == 0 ? 0.0 : -c.dt;
      us = wilson<Gd>(phi, ns, 0, t, g.layer, profile(aheadA(zs, tau, mv), mv));
      us = Gd::mul_dag(us, wilson<Gd>(phi, ns, 1, t, g.layer, profile(aheadB(0.0, tau, mv), mv)));
      if (q == 0) {
        store_link(us, U, 2, s, g.Vp);
#pragma unroll
        for (int k = 0; k < W; ++k) park[k * PITCH] = full_real(us, k);
      }
    }
    L u0;
#pragma unroll
    for (int k = 0; k < W; ++k) full_real(u0, k) = park[k * PITCH];
    A e = Gd::logi(Gd::mul_dag(u0, us));
    const double k = 1.0 / (c.a[2] * c.dt);
#pragma unroll
    for (int q = 0; q < NG; ++q) e.c[q] *= k;
    store_alg(e, E, 2, s, g.Vp);
    return;
  }
  const uint32_t s = (uint32_t)(z * g.layer) + t;
  auto get = [&](int nucleus, int p) -> L {
    L l;
#pragma unroll
    for (int k = 0; k < W; ++k) full_real(l, k) = v[(nucleus * W + k) * PITCH + p];
    return l;
  };
  // the layer's four profile weights, one per lane (an error function each, a fifth of the kernel
  // when every thread formed all four)
  const double zz = z * c.a[2], tau = threadIdx.x & 1 ? -c.dt : 0.0;
  const double w4 = profile(threadIdx.x & 2 ? aheadB(zz, tau, mv) : aheadA(zz, tau, mv), mv);
  const double lA[2] = {of_lane(w4, 0), of_lane(w4, 1)}, lB[2] = {of_lane(w4, 2), of_lane(w4, 3)};
  const bool flat = lA[0] == lA[1] && lB[0] == lB[1];
  L u[NL], u1[NL];   // at t0 and at t0 - dt
#pragma unroll 1
  for (int time = flat ? 0 : 1; time >= 0; --time) {
    const double wA = time ? lA[1] : lA[0], wB = time ? lB[1] : lB[0];
    __syncthreads();
    for (int p = threadIdx.x; p < 2 * PITCH; p += IC_BS) {
      const int nucleus = p >= PITCH ? 1 : 0, r = p - nucleus * PITCH;
      const int px = x0 + r % IC_RIM, py = y0 + r / IC_RIM;
      if (px > g.nt || py > g.nt) continue;   // beyond the rim of a short tile
      L V = wilson<Gd>(phi, ns, nucleus, (int64_t)(py % g.nt) * g.nt + px % g.nt, g.layer, nucleus ? wB : wA);
#pragma unroll
      for (int k = 0; k < W; ++k) v[(nucleus * W + k) * PITCH + r] = full_real(V, k);
    }
    __syncthreads();
    if (!has) continue;
    const int p = ty * IC_RIM + tx;
#pragma unroll
    for (int n = 0; n < NL; ++n) {
      const int pn = p + (i0 + n == 0 ? 1 : IC_RIM);
      const L D = Gd::mul_dag(get(0, p), get(0, pn));
      if (time) u1[n] = Gd::mul(D, Gd::mul_dag(get(1, p), get(1, pn)));
      else u[n] = Gd::mul(D, Gd::mul_dag(get(1, p), get(1, pn)));
    }
  }
  if (!has) return;
  const double k = 1.0 / (c.a[0] * c.dt);
#pragma unroll
  for (int n = 0; n < NL; ++n) {
    A e;
    if (!flat) {
      e = Gd::logi(Gd::mul_dag(u[n], u1[n]));
#pragma unroll
      for (int q = 0; q < NG; ++q) e.c[q] *= k;
    } else {   // zero, or NaN where the links are not finite
      const double o = full_real(u[n], 0) - full_real(u[n], 0);
#pragma unroll
      for (int q = 0; q < NG; ++q) e.c[q] = o;
    }
    store_link(u[n], U, i0 + n, s, g.Vp);
    store_alg(e, E, i0 + n, s, g.Vp);
  }
  if (z < g.nz - 1) {
    if (NL == 2 || i0 == 0) store_link(Gd::one(), U, 2, s, g.Vp);
    if (NL == 2 || i0 == 1) store_alg(Gd::alg_zero(), E, 2, s, g.Vp);
  }
}

template <typename Gd, typename T>
__global__ void k_ic_gauss(const T* __restrict__ U, const T* __restrict__ E, const T* __restrict__ F2,
                           double scale, T* __restrict__ rhoA, T* __restrict__ rhoB, Geom g, StepConst c) {
  constexpr int NG = Gd::NG;
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= g.V) return;
  const int64_t Vp = g.Vp;
  Site x;
  x.x = (int)(s % g.nt); x.y = (int)((s / g.nt) % g.nt); x.z = (int)(s / g.layer);
  typename Gd::Alg r = Gd::alg_zero();
  for (int i = 0; i < 3; ++i) {
    const int64_t sm = idx(g, shifted(g, x, i, -1));
    typename Gd::Link Um;
    load_link(Um, U, i, sm, Vp);
    typename Gd::Alg eh, em;
    load_alg(eh, E, i, s, Vp);
    load_alg(em, E, i, sm, Vp);
    if (F2) {
      typename Gd::Alg fh, fm;
      load_alg(fh, F2, i, s, Vp);
      load_alg(fm, F2, i, sm, Vp);
      for (int q = 0; q < NG; ++q) { eh.c[q] += scale * fh.c[q]; em.c[q] += scale * fm.c[q]; }
    }
    typename Gd::Alg tr = Gd::transport(Um, em);
    for (int q = 0; q < NG; ++q) r.c[q] += (eh.c[q] - tr.c[q]) / c.a[i];
  }
  typename Gd::Alg zero = Gd::alg_zero();
  const bool isB = x.z < g.nz / 2;
  store_alg(isB ? r : zero, rhoB, 0, s, Vp);
  store_alg(isB ? zero : r, rhoA, 0, s, Vp);
}

void launch_ic_phi(double* work, double* phi_out, int ng, const Geom& g, const StepConst& c, const McvConst& mv,
                   hipStream_t st) {
  const int nb = 2 * ng;
  const int64_t m = (int64_t)nb * g.layer;
  double* c1 = work + 2 * m;
  double* c2 = work + 4 * m;
  const int nt = g.nt, h = nt / 2 + 1;
  const DftConst k{nt, h, nb, c.a[0], mv.m_ir, mv.uv_cut};
  if (nt <= DFT_SMALL) {
    hipLaunchKernelGGL(k_dft_small, dim3(nb), dim3(DFT_SMALL_BS), 0, st, work, phi_out, k);
    return;
  }
  auto grid = [&](int lines) {
    return dim3((unsigned)((lines + DFT_LINES - 1) / DFT_LINES), (unsigned)((h + DFT_BS - 1) / DFT_BS), (unsigned)nb);
  };
  const dim3 block((unsigned)std::min(DFT_BS, (h + 63) / 64 * 64));   // whole wavefronts
  auto passes = [&](auto table) {
    constexpr bool TAB = decltype(table)::value;
    const unsigned lds = TAB ? (unsigned)(nt * sizeof(double2)) : 0;
    hipLaunchKernelGGL((k_dft<0, TAB>), grid(nt), block, lds, st, work, c1, k);
    hipLaunchKernelGGL((k_dft<1, TAB>), grid(h), block, lds, st, c1, c2, k);
    hipLaunchKernelGGL((k_dft<2, TAB>), grid(h), block, lds, st, c2, c1, k);
    hipLaunchKernelGGL((k_dft<3, TAB>), grid(nt), block, lds, st, c1, phi_out, k);
  };
  if (nt <= DFT_TABLE_MAX) passes(std::true_type{});
  else passes(std::false_type{});
}

template <typename G, typename T>
void launch_ic_fields(const double* phi, int ns, T* U, T* E, T* rhoA, T* rhoB, const Geom& g, const StepConst& c,
                      const McvConst& mv, hipStream_t st) {
  using Gd = typename GroupOf<G::NC, double>::type;
  const int bs = 256;
  const unsigned sb = (unsigned)((g.V + bs - 1) / bs);
  const unsigned nx = (unsigned)((g.nt + IC_TX - 1) / IC_TX), ny = (unsigned)((g.nt + IC_TY<Gd> - 1) / IC_TY<Gd>);
  // layers 0 .. nz - 1 and the seam, as many at a time as a grid's third dimension takes
  for (int z = 0; z <= g.nz; z += 32768)
    hipLaunchKernelGGL((k_ic_links<Gd, T>), dim3(nx, ny, (unsigned)std::min(32768, g.nz + 1 - z)), dim3(IC_BS), 0, st,
                       phi, ns, U, E, g, c, mv, z);
  // the semi-implicit scheme conserves D.(E + dt f1(U(t0), U(t0 - dt))) - rho instead;
  // its caller builds f1 and sets the charges through launch_gauss_charges
  if (c.scheme == 1) return;
  hipLaunchKernelGGL((k_ic_gauss<Gd, T>), dim3(sb), dim3(bs), 0, st, U, E, (const T*)nullptr, 0.0, rhoA, rhoB, g, c);
}

template <typename G, typename T>
void launch_gauss_charges(const T* U, const T* E, const T* F2, double scale, T* rhoA, T* rhoB, const Geom& g,
                          const StepConst& c, hipStream_t st) {
  using Gd = typename GroupOf<G::NC, double>::type;
  const int bs = 256;
  const unsigned sb = (unsigned)((g.V + bs - 1) / bs);
  hipLaunchKernelGGL((k_ic_gauss<Gd, T>), dim3(sb), dim3(bs), 0, st, U, E, F2, scale, rhoA, rhoB, g, c);
}

#define GL_GC_INST(G, T) \
  template void launch_gauss_charges<G, T>(const T*, const T*, const T*, double, T*, T*, const Geom&, const StepConst&, hipStream_t);
GL_GC_INST(Su2<double>, double)
GL_GC_INST(Su3<double>, double)
GL_GC_INST(Su2<float>, float)
GL_GC_INST(Su3<float>, float)
#define GL_IC_INST(G, T) \
  template void launch_ic_fields<G, T>(const double*, int, T*, T*, T*, T*, const Geom&, const StepConst&, \
                                       const McvConst&, hipStream_t);
GL_IC_INST(Su2<double>, double)
GL_IC_INST(Su3<double>, double)
GL_IC_INST(Su2<float>, float)
GL_IC_INST(Su3<float>, float)

}  // namespace gl
