// Group helpers of the reverse-mode (adjoint) kernels, double precision, host + device.
// Products of hermitian traceless matrices are formed from their components (AdjOps).
#pragma once
#include "group.h"

namespace gl {

// Products of algebra elements by components:
//   cross(x, y) = -i [X, Y],  cross^a = f^abc x^b y^c       (for i H forms: [i X, i Y] = -i cross)
//   sym(c0, c, x) = traceless part of {C, X}, C = c0 + c^a t^a:  2 c0 x^a + d^abc c^b x^c
// 50 and 62 multiply-adds for SU(3), a quarter of the two matrix products of a commutator.
template <typename G> struct AdjOps;
template <> struct AdjOps<Su2<double>> {
  using G = Su2<double>;
  static GL_HD G::Alg cross(const G::Alg& x, const G::Alg& y) {
    G::Alg z;
    z.c[0] = fmx(x.c[1], y.c[2], -x.c[2] * y.c[1]);
    z.c[1] = fmx(x.c[2], y.c[0], -x.c[0] * y.c[2]);
    z.c[2] = fmx(x.c[0], y.c[1], -x.c[1] * y.c[0]);
    return z;
  }
  // W = C + i S, both hermitian: c0, the components of C and those of S
  static GL_HD void split(const G::Link& w, double& c0, G::Alg& c, G::Alg& s) {
    c0 = w.q[0];
    c = G::alg_zero();
    s = G::proj(w);
  }
  static GL_HD G::Alg sym(double c0, const G::Alg&, const G::Alg& x) {
    G::Alg y;
    for (int k = 0; k < 3; ++k) y.c[k] = 2.0 * c0 * x.c[k];
    return y;
  }
};
template <> struct AdjOps<Su3<double>> {
  using G = Su3<double>;
  // f123 = 1, f147 = f246 = f257 = f345 = 1/2, f156 = f367 = -1/2, f458 = f678 = sqrt(3)/2
  static GL_HD G::Alg cross(const G::Alg& xx, const G::Alg& yy) {
    auto x = [&](int k) { return xx.c[k - 1]; };   // indices 1..8 as in the structure constants
    auto y = [&](int k) { return yy.c[k - 1]; };
    const double g = 0.86602540378443864676;
    const double h1 = 0.5 * x(1), h2 = 0.5 * x(2), h3 = 0.5 * x(3), h4 = 0.5 * x(4), h5 = 0.5 * x(5), h6 = 0.5 * x(6),
                 h7 = 0.5 * x(7), g8 = g * x(8);
    const double p38 = h3 + g8, q38 = g8 - h3;
    G::Alg z;
    z.c[0] = fmx(x(2), y(3), fmx(-x(3), y(2), fmx(h4, y(7), fmx(-h7, y(4), fmx(h6, y(5), -h5 * y(6))))));
    z.c[1] = fmx(x(3), y(1), fmx(-x(1), y(3), fmx(h4, y(6), fmx(-h6, y(4), fmx(h5, y(7), -h7 * y(5))))));
    z.c[2] = fmx(x(1), y(2), fmx(-x(2), y(1), fmx(h4, y(5), fmx(-h5, y(4), fmx(h7, y(6), -h6 * y(7))))));
    z.c[3] = fmx(h7, y(1), fmx(-h1, y(7), fmx(h6, y(2), fmx(-h2, y(6), fmx(h5, y(3), fmx(-p38, y(5), g * x(5) * y(8)))))));
    z.c[4] = fmx(h7, y(2), fmx(-h2, y(7), fmx(h1, y(6), fmx(-h6, y(1), fmx(p38, y(4), fmx(-h4, y(3), -g * x(4) * y(8)))))));
    z.c[5] = fmx(h2, y(4), fmx(-h4, y(2), fmx(h5, y(1), fmx(-h1, y(5), fmx(-h7, y(3), fmx(-q38, y(7), g * x(7) * y(8)))))));
    z.c[6] = fmx(h1, y(4), fmx(-h4, y(1), fmx(h2, y(5), fmx(-h5, y(2), fmx(h6, y(3), fmx(q38, y(6), -g * x(6) * y(8)))))));
    z.c[7] = g * (fmx(x(4), y(5), -x(5) * y(4)) + fmx(x(6), y(7), -x(7) * y(6)));
    return z;
  }
  static GL_HD void split(const G::Link& w, double& c0, G::Alg& c, G::Alg& s) {
    c0 = G::retr(w) * (1.0 / 3.0);
    c = G::alg_of_herm(w);
    s = G::proj(w);
  }
  // d118 = d228 = d338 = 1/sqrt(3), d448 = .. = d778 = -1/(2 sqrt(3)), d888 = -1/sqrt(3),
  // d146 = d157 = d256 = d344 = d355 = 1/2, d247 = d366 = d377 = -1/2
  static GL_HD G::Alg sym(double c0, const G::Alg& cc, const G::Alg& xx) {
    auto c = [&](int k) { return cc.c[k - 1]; };
    auto x = [&](int k) { return xx.c[k - 1]; };
    const double r = 0.57735026918962576451;
    const double h1 = 0.5 * c(1), h2 = 0.5 * c(2), h3 = 0.5 * c(3), h4 = 0.5 * c(4), h5 = 0.5 * c(5), h6 = 0.5 * c(6),
                 h7 = 0.5 * c(7), r8 = r * c(8);
    const double m = fmx(2.0, c0, r8);                      // rows 1-3
    const double n = fmx(2.0, c0, -0.5 * r8);               // rows 4-7
    const double rx8 = r * x(8), sx8 = -0.5 * rx8;
    G::Alg y;
    y.c[0] = fmx(m, x(1), fmx(c(1), rx8, fmx(h4, x(6), fmx(h6, x(4), fmx(h5, x(7), h7 * x(5))))));
    y.c[1] = fmx(m, x(2), fmx(c(2), rx8, fmx(-h4, x(7), fmx(-h7, x(4), fmx(h5, x(6), h6 * x(5))))));
    y.c[2] = fmx(m, x(3), fmx(c(3), rx8, fmx(h4, x(4), fmx(h5, x(5), fmx(-h6, x(6), -h7 * x(7))))));
    y.c[3] = fmx(n + h3, x(4), fmx(c(4), sx8, fmx(h1, x(6), fmx(h6, x(1), fmx(-h2, x(7), fmx(-h7, x(2), h4 * x(3)))))));
    y.c[4] = fmx(n + h3, x(5), fmx(c(5), sx8, fmx(h1, x(7), fmx(h7, x(1), fmx(h2, x(6), fmx(h6, x(2), h5 * x(3)))))));
    y.c[5] = fmx(n - h3, x(6), fmx(c(6), sx8, fmx(h1, x(4), fmx(h4, x(1), fmx(h2, x(5), fmx(h5, x(2), -h6 * x(3)))))));
    y.c[6] = fmx(n - h3, x(7), fmx(c(7), sx8, fmx(h1, x(5), fmx(h5, x(1), fmx(-h2, x(4), fmx(-h4, x(2), -h7 * x(3)))))));
    const double t = fmx(c(1), x(1), fmx(c(2), x(2), c(3) * x(3)));
    const double u = fmx(h4, x(4), fmx(h5, x(5), fmx(h6, x(6), h7 * x(7))));
    y.c[7] = fmx(2.0 * c0 - r8, x(8), r * (t - u));
    return y;
  }
};

template <typename A> GL_HD void axpy(A& y, double s, const A& x) {
  constexpr int NG = sizeof(y.c) / sizeof(y.c[0]);
#pragma unroll
  for (int k = 0; k < NG; ++k) y.c[k] += s * x.c[k];
}

// Reverse of U' = exp(i c E) U for the left-trivialised cotangent lam of U' (components): returns
//   ebar = c int_0^1 exp(-i s c E) Lam exp(i s c E) ds   and, in l,   exp(-i c E) Lam exp(i c E).
// With (ad b) y = -cross(b, y), b = c E / 2^m, the integral is the series
// sum_k (-ad b)^k Lam / (k+1)!, |ad b| <= rho <= 1, then m doublings
// I(2b) = (I(b) + e^-b I(b) e^b) / 2.  The series stops after the fewest terms N whose tail
// bound rho^(N+1) / (N+2)! is below 2^-15 / 16!, so its truncation error is below that
// relative for every field (18 terms at rho = 1); small fields (rho ~ 0.02-0.1) need 7-10.
// Since e^-b Lam e^b = Lam - (ad b) I, l costs one more product and no exponential when m = 0.
template <typename G>
GL_HD typename G::Alg dexp_reverse(const typename G::Alg& e, double c, const typename G::Alg& lam,
                                   typename G::Alg& l) {
  using Op = AdjOps<G>;
  constexpr int NG = G::NG;
  double n2 = 0.0;
#pragma unroll
  for (int k = 0; k < NG; ++k) n2 = fmx(e.c[k], e.c[k], n2);
  const double r = fabs(c) * sqrt(0.5 * n2);   // Frobenius norm of c E >= spectral norm
  int m = 0;
  double sc = 1.0;
  while (2.0 * r * sc > 1.0 && m < 60) { sc *= 0.5; ++m; }
  typename G::Alg b;
#pragma unroll
  for (int k = 0; k < NG; ++k) b.c[k] = c * sc * e.c[k];
  const double rho = 2.0 * r * sc;                             // bound on |ad b|
  const double tail_max = 3.0517578125e-05 / 20922789888000.0;   // 2^-15 / 16!
  int nt = 1;
  double tail = rho * rho / 6.0;                               // rho^(N+1) / (N+2)! at N = 1
  while (nt < 18 && tail > tail_max) {
    ++nt;
    tail *= rho / (double)(nt + 2);
  }
  typename G::Alg t = lam;
#pragma unroll 1
  for (int k = nt; k >= 1; --k) {
    const typename G::Alg z = Op::cross(b, t);
    const double w = 1.0 / (double)(k + 1);
#pragma unroll
    for (int q = 0; q < NG; ++q) t.c[q] = fmx(w, z.c[q], lam.c[q]);
  }
  if (m > 0) {
    typename G::Link X = G::expi(e, -c * sc);   // e^-b
#pragma unroll 1
    for (int q = 0; q < m; ++q) {
      const typename G::Alg y = G::transport_inv(X, t);   // e^-b I e^b
#pragma unroll
      for (int k = 0; k < NG; ++k) t.c[k] = 0.5 * (t.c[k] + y.c[k]);
      X = G::mul(X, X);
    }
    l = G::transport(G::expi(e, c), lam);   // (X has become e^-2^m b too, but every squaring doubled its error)
  } else {
    const typename G::Alg z = Op::cross(b, t);
#pragma unroll
    for (int k = 0; k < NG; ++k) l.c[k] = lam.c[k] + z.c[k];
  }
#pragma unroll
  for (int k = 0; k < NG; ++k) t.c[k] *= c;
  return t;
}

}  // namespace gl
