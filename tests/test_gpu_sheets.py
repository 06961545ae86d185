"""GPU parity of the multi-sheet initial conditions (glasma_init_mv_sheets: nuclei with
colour structure along the beam axis) against the FP64 oracle, and the evolution of
such a state; per-component bar 1e-10 as for the single sheet."""
import sys
import numpy as np
import pytest

import synth
from oracle import lattice, init_mv
from scipy.special import erfc
from _gpu import gpu, lattice_or_skip, to_comp, state_errs, mv_setup, new_lattice

pytestmark = gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


CASES = [
    (synth.Workload("su2-64x8x8-sheets", nc=2, nz=64, nt=8, mu=1.0, sigma=4.0, seed=1101), 5),
    (synth.Workload("su3-40x6x6-sheets", nc=3, nz=40, nt=6, mu=0.5, sigma=3.0, seed=1177), 4),
]


@pytest.mark.parametrize("w,ns", CASES, ids=[c[0].name for c in CASES])
def test_init_mv_sheets_matches_oracle_and_evolves(w, ns):
    pkg = lattice_or_skip()
    say("case:", w.name, "ns", ns)
    p, mv = mv_setup(w)
    rA, rB = synth.mv_sheet_charges(w.seed, w.nc, w.nt, w.mu, w.a_T, ns)
    st, _ = init_mv.initial_state(rA, rB, w.nz, p, mv)
    lat = new_lattice(pkg, w)
    lat.init_mv(rA, rB, m_ir=w.m_ir, uv_cut=w.uv_cut, sigma=w.sigma, zA=w.zA, zB=w.zB)
    errs = state_errs(lat.get_state(), st)
    say("init errs", errs)
    assert max(errs.values()) < 1e-10, errs
    o = lat.observables()
    assert o["gauss_rel"] < 1e-13 and o["unitarity"] < 1e-13
    worst = 0.0
    for s in range(20):
        st = lattice.leapfrog_step(st)
        lat.step(1)
        e = state_errs(lat.get_state(), st)
        worst = max(worst, max(e.values()))
        assert max(e.values()) < 1e-10, (s, e)
    say("per-component worst over 20 steps", worst)


@pytest.mark.parametrize("fp", [64, 32])
def test_identical_sheets_equal_one_sheet(fp):
    """rho_k = rho / ns for every sheet: the same state as the single sheet rho."""
    pkg = lattice_or_skip()
    w = synth.Workload("su3-32x8x8", nc=3, nz=32, nt=8, mu=0.5, sigma=2.0, seed=1203)
    ns = 3
    rA, rB = synth.mv_charges(w.seed, w.nc, w.nt, w.mu, w.a_T)
    one = new_lattice(pkg, w, fp=fp)
    one.init_mv(rA, rB, m_ir=w.m_ir, sigma=w.sigma)
    many = new_lattice(pkg, w, fp=fp)
    many.init_mv(np.repeat(rA[None] / ns, ns, 0), np.repeat(rB[None] / ns, ns, 0), m_ir=w.m_ir, sigma=w.sigma)
    a, b = one.get_state(), many.get_state()
    tol = 1e-12 if fp == 64 else 2e-6
    for k in ("U", "E", "rhoA", "rhoB"):
        ref = np.asarray(a[k])
        d = np.abs(np.asarray(b[k]) - ref).max() / max(np.abs(ref).max(), 1e-300)
        say(fp, k, d)
        assert d < tol, (k, d)


def test_sheet_arguments_are_checked():
    pkg = lattice_or_skip()
    w = synth.Workload("su3-4x8x8", nc=3, nz=4, nt=8, mu=0.5, sigma=1.0, seed=5)
    lat = new_lattice(pkg, w, fp=32)
    # second link buffer: 3 * 12 * 256 floats = 36864 bytes holds 4 sheets of 2 * 8 * 64 doubles
    rA, rB = synth.mv_sheet_charges(w.seed, 3, 8, 0.5, w.a_T, 4)
    lat.init_mv(rA, rB, sigma=1.0)
    rA, rB = synth.mv_sheet_charges(w.seed, 3, 8, 0.5, w.a_T, 5)
    with pytest.raises(pkg.GlasmaError, match="too many sheets"):
        lat.init_mv(rA, rB, sigma=1.0)
    with pytest.raises(ValueError):
        lat.init_mv(rA, rB[:2], sigma=1.0)


@pytest.mark.parametrize("nc,nz,nt,ns", [(2, 64, 15, 1), (3, 64, 16, 2), (3, 64, 17, 1), (2, 64, 33, 3), (3, 64, 2, 1)])
def test_init_tile_edges(nc, nz, nt, ns):
    """The initial links come in tiles of 16 x 16 transverse sites with a rim on +x and +y:
    lattices of one short, one full and several tiles, and the smallest.  Nuclei narrow
    enough that some layers have equal profiles at both times (farther than 38 sigma ahead of
    one nucleus and 8.4 sigma behind the other) and others do not.  Links, E and charges
    against the oracle to 1e-10, as the test above."""
    pkg = lattice_or_skip()
    w = synth.Workload(f"su{nc}-{nz}x{nt}-sheets{ns}", nc=nc, nz=nz, nt=nt, mu=0.2, sigma=0.35, seed=820 + nt)
    print("case: initial tiles", w.name, flush=True)
    p, mv = mv_setup(w)
    if ns == 1:
        rA, rB = synth.mv_charges(w.seed, nc, nt, w.mu, w.a_T)
    else:
        rA, rB = synth.mv_sheet_charges(w.seed, nc, nt, w.mu, w.a_T, ns)
    st, _ = init_mv.initial_state(rA, rB, nz, p, mv)
    lat = new_lattice(pkg, w)
    lat.init_mv(rA, rB, m_ir=w.m_ir, uv_cut=w.uv_cut, sigma=w.sigma, zA=w.zA, zB=w.zB)
    errs = state_errs(lat.get_state(), st)
    print(" ", errs, flush=True)
    assert max(errs.values()) < 1e-10, errs


def test_initial_field_of_whole_matrices():
    """The rounding of E(t0 - dt/2) after 8 sheets, SU(3): rms error over all transverse links against
    extended precision, compared with that of the same group operations on whole matrices (the library's
    own, run on the host; same sequence of exponentials and products, profiles in double as well).  The
    fields are weak (|phi| ~ 0.05 a sheet), so that the matrices' rounding decides and not that of phi
    (3e-16 of E).  The device's error function adds its own rounding: half a unit 2^-53 rms in the two
    profiles that E is the difference of, over dt times the profile's density at the centre.  Bound: both
    together, and a tenth.  With intermediate matrices cut to two rows the error is half as large again."""
    pkg = lattice_or_skip()
    mp = pytest.importorskip("mpmath")
    if np.finfo(np.longdouble).eps > 2.0 ** -60:
        pytest.skip("no extended precision here")
    nc, nz, nt, ns, a_T, dt, m = 3, 16, 16, 8, 4.0, 0.5, 0.2
    sigma, zA, zB = 3.0, 9.0, 6.0
    say("case: rounding of the initial field", nz, nt, ns)
    g = synth.rng(951)
    rho = g.standard_normal((2, ns, 8, nt, nt)) * 0.1 / (a_T * np.sqrt(ns))
    lat = pkg.Lattice(nc=nc, nz=nz, nt=nt, a_T=a_T, dt=dt)
    lat.init_mv(rho[0], rho[1], m_ir=m, sigma=sigma, zA=zA, zB=zB)
    got = lat.get_state()["E"][:2].reshape(2, 8, nz, nt, nt)

    ld = np.longdouble
    pi = ld("3.14159265358979323846264338327950288")
    ph = (np.outer(np.arange(nt), np.arange(nt)) % nt).astype(ld) * 2 * pi / nt
    W = np.cos(ph) - 1j * np.sin(ph)
    s2 = (ld(2) / ld(a_T) * np.sin(pi * np.arange(nt, dtype=ld) / nt)) ** 2
    filt = 1 / (s2[:, None] + s2[None, :] + ld(m) * ld(m))
    phi = np.real(np.conj(W) @ ((W @ rho.astype(ld) @ W) * filt) @ np.conj(W)) / (nt * nt)   # (2, ns, 8, y, x)
    with mp.workdps(30):
        wt = np.array([[[ld(mp.nstr(mp.erfc(d / (mp.sqrt(2) * sigma)) / 2, 25)) for d in
                         (-(z - zA + tau) if n == 0 else z - zB - tau for z in range(nz))] for tau in (0.0, -dt)]
                       for n in range(2)])                                    # (nucleus, time, z)
    r3 = 1 / np.sqrt(ld(3))
    t = np.zeros((8, 3, 3), np.clongdouble)
    for a, (i, j) in enumerate([(0, 1), (0, 1), (0, 0), (0, 2), (0, 2), (1, 2), (1, 2), (2, 2)]):
        if a == 2:
            t[a] = np.diag([1, -1, 0]) / 2
        elif a == 7:
            t[a] = np.diag([r3, r3, -2 * r3]) / 2
        elif a in (0, 3, 5):
            t[a, i, j] = t[a, j, i] = 0.5
        else:
            t[a, i, j], t[a, j, i] = -0.5j, 0.5j
    comps = lambda h: np.stack([2 * np.real(sum(t[a][i, j] * h[..., j, i] for i in range(3) for j in range(3)))
                                for a in range(8)], -1)
    dag = lambda x: np.conj(np.swapaxes(x, -1, -2))

    def proj(x):
        y = (x - dag(x)) / 2j
        return y - np.trace(y, axis1=-2, axis2=-1)[..., None, None] / 3 * np.eye(3)

    def expi(h):
        x, out = 1j * h / 64, np.eye(3) + 0 * h
        for n in range(18, 0, -1):
            out = np.eye(3) + x @ out / n
        for _ in range(6):
            out = out @ out
        return out

    def log(w):
        h = proj(w)
        for _ in range(6):
            e = expi(-h / 2)
            h = h + proj(e @ w @ e)
        return h

    # extended precision, and the host's group operations in double, the profiles too: V (z, y, x)
    wd = np.array([[0.5 * erfc(np.array([-(z - zA + tau) if n == 0 else z - zB - tau for z in range(nz)]) /
                               (1.4142135623730951 * sigma)) for tau in (0.0, -dt)] for n in range(2)])
    weight = lambda v, n, time, k: np.clip(ns * v[n, time] - k, 0, 1)
    link = lambda r: r.reshape(-1, 18)
    hmul = lambda a, b: pkg.host_group_op(3, 64, 6, np.concatenate([a, b], 1), 18)

    def hdag(r):
        q = r.reshape(-1, 3, 3, 2).transpose(0, 2, 1, 3).copy()
        q[..., 1] *= -1
        return link(np.ascontiguousarray(q))

    U, H = {}, {}
    for time in range(2):
        D, F = [None, None], [None, None]
        for n in range(2):
            V = F_ = None
            for k in range(ns):
                lam = weight(wt, n, time, k)
                mat = np.einsum("ayx,aij->yxij", phi[n, k], t)
                e = expi(-lam[:, None, None, None, None] * mat[None])
                V = e if V is None else V @ e
                c = np.broadcast_to(phi[n, k].astype(float).transpose(1, 2, 0), (nz, nt, nt, 8)).reshape(-1, 8)
                s = np.repeat(-weight(wd, n, time, k), nt * nt)[:, None]
                x = pkg.host_group_op(3, 64, 0, np.concatenate([s, c], 1), 18)
                F_ = x if F_ is None else np.where(s < 0, hmul(F_, x), F_)
            D[n] = [V @ dag(np.roll(V, -1, axis=2 - i)) for i in range(2)]
            F4 = F_.reshape(nz, nt, nt, 18)
            F[n] = [hmul(F_, hdag(link(np.ascontiguousarray(np.roll(F4, -1, axis=2 - i))))) for i in range(2)]
        U[time] = [D[0][i] @ D[1][i] for i in range(2)]
        H[time] = [hmul(F[0][i], F[1][i]) for i in range(2)]
    ref = np.stack([comps(log(U[0][i] @ dag(U[1][i]))) for i in range(2)]) / (ld(a_T) * ld(dt))
    host = np.stack([pkg.host_group_op(3, 64, 1, hmul(H[0][i], hdag(H[1][i])), 8).reshape(nz, nt, nt, 8)
                     for i in range(2)]) * (1.0 / (a_T * dt))
    got = got.transpose(0, 2, 3, 4, 1)
    size = np.sqrt(np.mean(ref ** 2))
    eg, eh = (float(np.sqrt(np.mean((x - ref) ** 2)) / size) for x in (got, host))
    say("  rms error of E / rms E: kernel", eg, "whole matrices on the host", eh)
    profiles = np.sqrt(2) * 2.0 ** -54 / (dt / (np.sqrt(2 * np.pi) * sigma))
    assert eg <= 1.1 * np.hypot(eh, profiles)


@pytest.mark.parametrize("nc", [2, 3])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_non_finite_charges_reach_every_layer(nc, value):
    """One non-finite charge makes phi of its colour non-finite everywhere (a sum over all modes), so U and
    E(t0 - dt/2) of every transverse link are, also in layers that the profiles of both times reach
    equally, where E is not formed from a logarithm."""
    pkg = lattice_or_skip()
    nz, nt = 64, 16
    say("case: non-finite charge", nc, value)
    rho = np.full((nc * nc - 1, nt, nt), 0.01)
    bad = rho.copy()
    bad[1, 3, 5] = value
    lat = pkg.Lattice(nc=nc, nz=nz, nt=nt)
    lat.init_mv(bad, rho, sigma=0.35)
    got = lat.get_state()
    for k in ("U", "E"):
        f = got[k][:2].reshape(2, -1, nz, nt * nt)
        assert not np.isfinite(f).all(axis=1).any(), k
    lat.init_mv(rho, rho, sigma=0.35)
    assert all(np.isfinite(lat.get_state()[k]).all() for k in ("U", "E", "rhoA", "rhoB"))


@pytest.mark.parametrize("nc,nz", [(2, 32768), (3, 32770)])
def test_init_of_more_layers_than_a_grid_takes(nc, nz):
    """The initial links come in launches of at most 32768 layers: the seam alone in the second (nz =
    32768), two layers and the seam in the second (32770).  Nucleus A sits at the end, so that fields cross
    from one launch into the next; links, E and charges against the oracle to 1e-10."""
    pkg = lattice_or_skip()
    w = synth.Workload(f"su{nc}-{nz}x2", nc=nc, nz=nz, nt=2, mu=0.5, sigma=2.0, seed=860 + nc, zA=nz - 6.0, zB=40.0)
    say("case: layers", w.name)
    p, mv = mv_setup(w)
    rA, rB = synth.mv_charges(w.seed, nc, 2, w.mu, w.a_T)
    st, _ = init_mv.initial_state(rA, rB, nz, p, mv)
    lat = new_lattice(pkg, w)
    lat.init_mv(rA, rB, m_ir=w.m_ir, uv_cut=w.uv_cut, sigma=w.sigma, zA=w.zA, zB=w.zB)
    errs = state_errs(lat.get_state(), st)
    say(" ", errs)
    assert max(errs.values()) < 1e-10, errs
