"""CPU checks of the reverse pass's algebra (csrc/adjoint.h): a small program over the header, compiled for
the host alone, against the matrices that the components stand for."""
import subprocess

import numpy as np
import pytest

from oracle import su
from test_sweep_order import build

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "adjoint.h"
using namespace gl;
template <typename A> static A rd() {
  A a;
  for (double& x : a.c) if (scanf("%lf", &x) != 1) exit(1);
  return a;
}
template <typename A> static void wr(const A& a) { for (double x : a.c) printf("%.17g ", x); }
template <typename G> static void run(int op, int n) {
  using Op = AdjOps<G>;
  using A = typename G::Alg;
  for (int i = 0; i < n; ++i) {
    if (op == 0) {          // reverse of the exponential: c, e, lam -> integral, transported lam
      double c;
      if (scanf("%lf", &c) != 1) exit(1);
      const A e = rd<A>(), lam = rd<A>();
      A l;
      const A r = dexp_reverse<G>(e, c, lam, l);
      wr(r);
      wr(l);
    } else {                // w = exp(i e): x, y -> cross(x, y), c0, C, S of w, sym(C, x)
      const A e = rd<A>(), x = rd<A>(), y = rd<A>();
      double c0;
      A c, s;
      Op::split(G::expi(e, 1.0), c0, c, s);
      wr(Op::cross(x, y));
      printf("%.17g ", c0);
      wr(c);
      wr(s);
      wr(Op::sym(c0, c, x));
    }
    printf("\n");
  }
}
int main(int, char** v) {
  const int op = atoi(v[2]), n = atoi(v[3]);
  if (v[1][0] == '2') run<Su2<double>>(op, n);
  else run<Su3<double>>(op, n);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = build(tmp_path_factory.mktemp("adjoint"), "algebra", SOURCE)

    def run(nc, op, rows):
        text = "\n".join(" ".join(repr(float(x)) for x in r) for r in rows)
        out = subprocess.run([exe, str(nc), str(op), str(len(rows))], input=text, capture_output=True, text=True, check=True)
        return np.array([[float(x) for x in line.split()] for line in out.stdout.splitlines()])

    return run


@pytest.mark.parametrize("nc", [2, 3])
def test_products_by_components(program, nc):
    """cross, split and sym against commutators, hermitian parts and anticommutators of matrices; sums of at
    most 20 products of numbers of order 1: 1e-14."""
    ng = nc * nc - 1
    g = np.random.default_rng(11)
    e, x, y = g.standard_normal((3, 40, ng)) * np.array([0.7, 1.0, 1.0])[:, None, None]
    out = program(nc, 1, np.concatenate([e, x, y], 1))
    E, X, Y = (su.from_components(a, nc) for a in (e, x, y))
    W = su.expi(E)
    C, S = (W + su.dag(W)) / 2, (W - su.dag(W)) / 2j
    eye = np.eye(nc)
    tr = lambda m: np.trace(m, axis1=-2, axis2=-1)[..., None, None] / nc * eye
    ref = [su.to_components(-1j * (X @ Y - Y @ X)), np.trace(C, axis1=-2, axis2=-1).real[:, None] / nc,
           su.to_components(C - tr(C)), 2 * su.to_components(S - tr(S)) / 2]
    an = C @ X + X @ C
    ref.append(su.to_components(an - tr(an)))
    got = np.split(out, np.cumsum([ng, 1, ng, ng]), axis=1)
    for name, a, b in zip(("cross", "c0", "C", "S", "sym"), got, ref):
        assert np.abs(a - b).max() < 1e-14, (name, np.abs(a - b).max())


@pytest.mark.parametrize("nc", [2, 3])
def test_reverse_of_the_exponential(program, nc):
    """Both results of the reverse of U' = exp(i c E) U in 40 digits, fields |c E| (Frobenius) from 0.02
    to 20, below, above and far above the bound of the series alone.  Relative error of the transported
    cotangent, in units of 2^-53: 8 of its own products, and of the exponential 4 |c E| for SU(2) (its angle's
    rounding, turned twice), 10 |c E| and 16 for SU(3) (14 terms, each halving doubled back); of the
    integral 16 and 40 |c E| (every doubling doubles what it adds up)."""
    mp = pytest.importorskip("mpmath")
    mp.mp.dps = 40
    ng = nc * nc - 1
    t = [mp.matrix(m.tolist()) for m in su.generators(nc)]
    if nc == 3:
        t[7] = mp.diag([1, 1, -2]) / (2 * mp.sqrt(3))
    comps = lambda m: [2 * mp.re(sum((t[a] * m)[i, i] for i in range(nc))) for a in range(ng)]
    g = np.random.default_rng(3)
    for h in (0.02, 0.45, 0.6, 1.0, 2.0, 5.0, 20.0):
        rows = []
        for _ in range(12):
            e, lam = g.standard_normal((2, ng))
            rows.append(np.concatenate([[2.0], e * h / 2.0 / np.sqrt(0.5 * np.sum(e ** 2)), lam]))
        out = program(nc, 0, rows)
        err = np.zeros(2)
        for row, got in zip(rows, out):
            E, lam = mp.zeros(nc), mp.zeros(nc)
            for a in range(ng):
                E += mp.mpf(row[1 + a]) * t[a]
                lam += mp.mpf(row[1 + ng + a]) * t[a]
            w, V = mp.eighe(E)
            M = V.transpose_conj() * lam * V
            r, l = mp.zeros(nc), mp.zeros(nc)
            for i in range(nc):
                for j in range(nc):
                    d = 2 * (w[j] - w[i])
                    l[i, j] = M[i, j] * mp.expj(d)
                    r[i, j] = 2 * M[i, j] * ((mp.expj(d) - 1) / (1j * d) if abs(d) > mp.mpf(10) ** -25 else 1)
            for q, m in enumerate((r, l)):
                ref = comps(V * m * V.transpose_conj())
                d = mp.sqrt(sum((mp.mpf(got[q * ng + a]) - ref[a]) ** 2 for a in range(ng)))
                err[q] = max(err[q], float(d / mp.sqrt(sum(x * x for x in ref))) * 2.0 ** 53)
        bound = (16 + 40 * h, 8 + 4 * h if nc == 2 else 24 + 10 * h)
        assert err[0] <= bound[0] and err[1] <= bound[1], (h, err, bound)
