"""Boost-invariant Glasma (Sec. 2, eqs. glasma_ic1/2, LC_gauge1).

glasma_bi_fields against the oracle's tau = 0+ fields, element by element.

Boost-invariant limit: at mid-rapidity, shortly after thin
nuclei have passed through each other, the 3+1D Glasma carries the longitudinal fields of
the tau = 0+ boost-invariant initial condition of the same nuclei (oracle.glasma_bi):
p_T = eps_0 and p_L < 0 (flux tubes).  The nuclei must be resolved by the longitudinal
lattice and thin against 1/Q_s, so the lattice is fine along z: a_T = 16 a_L, dilute MV
charges (mu a_T = 1.4, m a_T = 0.8), sigma = 8, 4, 2 a_L.  The whole GPU pipeline (initial
conditions, CPIC, semi-implicit scheme at dt = a_L, observables, boost-invariant fields);
expected: p_T(z_c)/eps_0 rises towards 1 as sigma shrinks and p_L turns negative."""
import sys
import numpy as np
import pytest

import synth
from oracle import su, lattice, init_mv, glasma_bi
from _gpu import gpu, lattice_or_skip

pytestmark = gpu


@pytest.mark.parametrize("nc,nt,ns", [(2, 12, 1), (3, 10, 1), (3, 16, 3)])
def test_bi_fields_match_oracle(nc, nt, ns):
    pkg = lattice_or_skip()
    print("case: boost-invariant fields nc", nc, "nt", nt, "sheets", ns, flush=True)
    a_T, m = 4.0, 0.2
    if ns == 1:
        rA, rB = synth.mv_charges(91, nc, nt, 0.6, a_T)
    else:
        rA, rB = synth.mv_sheet_charges(91, nc, nt, 0.6, a_T, ns)
    p = lattice.Params(nc=nc, a_T=a_T, a_L=1.0, dt=0.5)
    mv = init_mv.MVParams(m_ir=m, uv_cut=0.0)
    aA = glasma_bi.transverse_alpha(glasma_bi.wilson_behind(rA, p, mv), a_T)
    aB = glasma_bi.transverse_alpha(glasma_bi.wilson_behind(rB, p, mv), a_T)
    Ez, Bz = glasma_bi.bi_fields(aA, aB)
    e0 = glasma_bi.bi_energy(aA, aB)
    got = pkg.boost_invariant_fields(nc, nt, rA, rB, a_T=a_T, m_ir=m)
    for name, ref in (("Ez", Ez), ("Bz", Bz)):
        r = np.moveaxis(su.to_components(ref), -1, 0)
        g = got[name].cpu().numpy()
        err = np.abs(g - r).max() / np.abs(r).max()
        print(" ", name, "max rel err", err, flush=True)
        assert err < 1e-11, (name, err)
    np.testing.assert_allclose([got["eps0"], got["EL2_half"], got["BL2_half"]], e0, rtol=1e-11)


def scan(pkg, sigma, scheme=1, dt=1.0):
    nc, nt, nz, aT = 3, 32, 96, 16.0
    m, mu, zA, zB = 0.8 / aT, 1.4 / aT, 72.0, 24.0
    rA, rB = synth.mv_charges(77, nc, nt, mu, aT)
    e0 = pkg.boost_invariant_fields(nc, nt, rA, rB, a_T=aT, m_ir=m)["eps0"]
    lat = pkg.Lattice(nc=nc, nz=nz, nt=nt, a_T=aT, a_L=1.0, dt=dt, fp=64, scheme=scheme, max_iter=300,
                      tol=1e-12)
    lat.init_mv(rA, rB, m_ir=m, uv_cut=0.0, sigma=sigma, zA=zA, zB=zB)
    t_c, z_c = 0.5 * (zA - zB), int(0.5 * (zA + zB))
    s_c = int(round(t_c / dt))
    per = int(round(2 / dt))
    lat.step(s_c)
    pt, pl = [], []
    for _ in range(10):
        lat.step(per)
        sl = lat.observables()["tmunu_z"]
        pt.append(sl[2][z_c] / e0)
        pl.append(sl[1][z_c] / sl[0][z_c])
    return np.array(pt), np.array(pl)


def test_thin_nuclei_approach_the_boost_invariant_glasma():
    pkg = lattice_or_skip()
    peaks, mins = [], []
    for sig in (8.0, 4.0, 2.0):
        print("case: boost-invariant limit, sigma", sig, flush=True)
        pt, pl = scan(pkg, sig)
        print("  p_T/eps_0", np.round(pt, 3), "p_L/eps", np.round(pl, 3), flush=True)
        peaks.append(pt.max())
        mins.append(pl.min())
    assert peaks[0] < peaks[1] < peaks[2], peaks
    assert abs(peaks[2] - 1.0) < 0.15, peaks
    assert mins[0] > 0.0 and mins[2] < -0.5, mins


@pytest.mark.parametrize("nt", [2, 3, 31, 32, 33, 64, 129, 258, 513, 2050])
def test_transverse_field_sizes(nt):
    """The DFT passes of the transverse Poisson equation at the edges of their forms: one
    work-group per plane (up to 32), staged lines (from 33; sums of one, two and three chunks
    of 256 terms; one and several blocks of outputs), lines beyond the phase table (2050).
    One colour per nucleus, SU(2): alpha^i_N = 2 sin(d_i phi_N / 2) / a_T in closed form, and
    E_z^3 is the site average of alpha_A^i alpha_B^i, with phi from numpy's FFT.  Sums of nt
    terms of rounding 2^-53 each and their products stay far below 1e-11 of the largest."""
    pkg = lattice_or_skip()
    print("case: transverse field, nt", nt, flush=True)
    a_T, m, cut = 4.0, 0.2, 0.6   # |k~| up to 0.71: part of the modes is cut, at nt = 2 one
    g = synth.rng(500 + nt)
    rho = np.zeros((2, 3, nt, nt))
    rho[0, 0], rho[1, 1] = g.standard_normal((2, nt, nt)) * 0.1
    k2 = init_mv.ktilde2(nt, a_T)
    filt = np.where(np.sqrt(k2) <= cut, 1.0 / (k2 + m * m), 0.0)
    phi = [np.real(np.fft.ifft2(np.fft.fft2(rho[n, n]) * filt)) for n in range(2)]
    ez = np.zeros((nt, nt))
    for ax in (-1, -2):
        al = [2.0 * np.sin((np.roll(p, -1, axis=ax) - p) / 2) / a_T for p in phi]
        ez += 0.5 * (al[0] * al[1] + np.roll(al[0] * al[1], 1, axis=ax))
    got = pkg.boost_invariant_fields(2, nt, rho[0], rho[1], a_T=a_T, m_ir=m, uv_cut=cut)["Ez"].cpu().numpy()
    err = np.abs(got[2] - ez).max() / max(np.abs(ez).max(), 1e-300)
    print("  max error / max", err, flush=True)
    assert err < 1e-11 and np.abs(got[:2]).max() <= 1e-11 * np.abs(ez).max()


@pytest.mark.parametrize("nt", [32, 192, 256])
def test_transverse_field_rounding(nt):
    """The rounding of phi: one colour per nucleus with |phi| ~ 40, so that phi's error decides that of
    E_z (closed form as above), against phi in extended precision.  Sums of nt products in blocks of b
    leave a relative rms error of a few times (sqrt(b) + sqrt(nt / b)) / 2 units of 2^-53 at most, where
    plain sums leave sqrt(nt) / 2 in each of four passes: below 6 units for the blocks, about 8 and 9
    units for plain sums of 192 and 256.  Bound: the error that independent errors of 6 units in phi
    and 2 in the links' angles would make."""
    pkg = lattice_or_skip()
    print("case: transverse field rounding, nt", nt, flush=True)
    if np.finfo(np.longdouble).eps > 2.0 ** -60:
        pytest.skip("no extended precision here")
    a_T, m = 4.0, 0.2
    g = synth.rng(900 + nt)
    rho = np.zeros((2, 3, nt, nt))
    rho[0, 0], rho[1, 1] = g.standard_normal((2, nt, nt)) * 10.0
    k = np.arange(nt, dtype=np.longdouble)
    pi = np.longdouble("3.14159265358979323846264338327950288")
    ph = (np.outer(np.arange(nt), np.arange(nt)) % nt).astype(np.longdouble) * 2 * pi / nt
    W = np.cos(ph) - 1j * np.sin(ph)
    s2 = (np.longdouble(2) / np.longdouble(a_T) * np.sin(pi * k / nt)) ** 2
    filt = 1 / (s2[:, None] + s2[None, :] + np.longdouble(m) * np.longdouble(m))
    phi = [np.real(np.conj(W) @ ((W @ r.astype(np.longdouble) @ W) * filt) @ np.conj(W)) / (nt * nt) for r in (rho[0, 0], rho[1, 1])]

    def field(p):
        ez = 0
        for ax in (-1, -2):
            al = [2 * np.sin((np.roll(q, -1, axis=ax) - q) / 2) / np.longdouble(a_T) for q in p]
            ez = ez + 0.5 * (al[0] * al[1] + np.roll(al[0] * al[1], 1, axis=ax))
        return ez

    ref = field(phi)
    rms = [np.sqrt(np.mean(q ** 2)) for q in phi]
    off = [q + 2.0 ** -53 * np.sqrt(6.0 ** 2 + 2.0 ** 2) * r * g.standard_normal((nt, nt)) for q, r in zip(phi, rms)]
    bound = np.sqrt(np.mean((field(off) - ref) ** 2))
    got = pkg.boost_invariant_fields(2, nt, rho[0], rho[1], a_T=a_T, m_ir=m)["Ez"].cpu().numpy()[2]
    err = np.sqrt(np.mean((got - ref) ** 2))
    print("  |phi|", float(rms[0]), "rms error", float(err), "bound", float(bound), flush=True)
    assert err <= bound


@pytest.mark.parametrize("nt", [27, 47, 97])
@pytest.mark.parametrize("axis", [-1, -2])
def test_cut_between_the_roundings_of_a_mode(nt, axis):
    """A cut at a mode's |k~| can lie between sin(pi k / nt) and sin(pi (nt - k) / nt) as rounded (13 to 32
    units of 2^-53 apart here): one of +-k is then left, so half of the mode, along x and along y
    alike.  Plane waves of the lowest mode, one colour per nucleus, closed form as above."""
    pkg = lattice_or_skip()
    print("case: cut between roundings, nt", nt, "axis", axis, flush=True)
    a_T, m = 4.0, 0.2
    pi = np.longdouble("3.14159265358979323846264338327950288")
    s = [np.sin(pi * np.longdouble(1.0 / nt)), np.sin(pi * (1 - np.longdouble((nt - 1) / nt)))]
    cut = float(np.longdouble(2) / np.longdouble(a_T) * (s[0] + s[1]) / 2)
    ang = 2 * np.pi * np.arange(nt) / nt
    wave = [np.cos(ang), np.sin(ang)]
    rho = np.zeros((2, 3, nt, nt))
    for n in range(2):
        rho[n, n] = 0.1 * (wave[n][None, :] if axis == -1 else wave[n][:, None])
    phi = [0.5 * rho[n, n] / ((2 / a_T * np.sin(np.pi / nt)) ** 2 + m * m) for n in range(2)]
    al = [2.0 * np.sin((np.roll(p, -1, axis=axis) - p) / 2) / a_T for p in phi]
    ez = 0.5 * (al[0] * al[1] + np.roll(al[0] * al[1], 1, axis=axis))
    got = pkg.boost_invariant_fields(2, nt, rho[0], rho[1], a_T=a_T, m_ir=m, uv_cut=cut)["Ez"].cpu().numpy()[2]
    err = np.abs(got - ez).max() / np.abs(ez).max()
    print("  max error / max", err, flush=True)
    assert err < 1e-11
