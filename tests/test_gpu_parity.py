"""GPU parity: the HIP library (through the C-ABI) against the FP64 oracle on the same
seeded inputs.  Per field component the bar is |d| <= 1e-10 max(|ref|, RMS of the
field) over the first 20 steps; gauge-invariant observables 1e-8 relative over the
full run (the dynamics is chaotic, so round-off differences grow)."""
import sys
import numpy as np
import pytest

import synth
from oracle import lattice, init_mv, observables, su
from _gpu import (gpu, lattice_or_skip, to_comp, from_comp, field_err, state_errs, mv_setup,
                  new_lattice)

pytestmark = gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _obs_close(go, oo, tol):
    sl_ref = oo["tmunu_z"]
    scale = np.abs(sl_ref).max(axis=1, keepdims=True)
    err_sl = np.max(np.abs(go["tmunu_z"] - sl_ref) / scale)
    err_H = abs(go["energy"] - oo["energy"]) / abs(oo["energy"])
    assert err_sl < tol and err_H < tol, (err_sl, err_H)
    return err_sl, err_H


def test_leapfrog_su2_fp64_small_workload():
    """SU(2) FP64, 64 x 8 x 8, MV nuclei, 100 steps (per-component parity over 20)."""
    pkg = lattice_or_skip()
    w = synth.SMALL_SU2
    say("case: su2 fp64 64x8x8 leapfrog, seed", w.seed)
    p, mv = mv_setup(w)
    rA, rB = synth.mv_charges(w.seed, w.nc, w.nt, w.mu, w.a_T)
    st, _ = init_mv.initial_state(rA, rB, w.nz, p, mv)
    lat = new_lattice(pkg, w)
    lat.init_state(*to_comp(st), step0=0)
    worst = 0.0
    for s in range(20):
        st = lattice.leapfrog_step(st)
        lat.step(1)
        errs = state_errs(lat.get_state(), st)
        worst = max(worst, max(errs.values()))
        assert max(errs.values()) < 1e-10, (s, errs)
    say("per-component worst over 20 steps", worst)
    for s in range(20, w.steps):
        if s % 10 == 0:
            _obs_close(lat.observables(), observables.observables(st), 1e-8)
        st = lattice.leapfrog_step(st)
        lat.step(1)
    go = lat.observables()
    err = _obs_close(go, observables.observables(st), 1e-8)
    say("observables at step 100", err)
    assert go["gauss_rel"] < 1e-12


@pytest.mark.parametrize("nc", [2, 3])
def test_init_mv_matches_oracle(nc):
    pkg = lattice_or_skip()
    w = synth.SMALL_SU2 if nc == 2 else synth.Workload("su3-40x6x6", nc=3, nz=40, nt=6, mu=0.5,
                                                        sigma=3.0, seed=77)
    say("case: init_mv nc", nc, "dims", w.nz, w.nt)
    p, mv = mv_setup(w)
    rA, rB = synth.mv_charges(w.seed, w.nc, w.nt, w.mu, w.a_T)
    st, _ = init_mv.initial_state(rA, rB, w.nz, p, mv)
    lat = new_lattice(pkg, w)
    lat.init_mv(rA, rB, m_ir=w.m_ir, uv_cut=w.uv_cut, sigma=w.sigma, zA=w.zA, zB=w.zB)
    errs = state_errs(lat.get_state(), st)
    say("init errs", errs)
    assert max(errs.values()) < 1e-10, errs
    o = lat.observables()
    assert o["gauss_rel"] < 1e-13 and o["unitarity"] < 1e-13


def test_leapfrog_su3_fp64_ragged_tiles():
    """SU(3) FP64 on 24 x 10 x 10 (2400 sites: 9 full blocks of 256 + a ragged tail)."""
    pkg = lattice_or_skip()
    w = synth.Workload("su3-24x10x10", nc=3, nz=24, nt=10, mu=0.5, sigma=2.0, seed=91)
    say("case: su3 fp64 24x10x10")
    p, mv = mv_setup(w)
    rA, rB = synth.mv_charges(w.seed, 3, w.nt, w.mu, w.a_T)
    st, _ = init_mv.initial_state(rA, rB, w.nz, p, mv)
    lat = new_lattice(pkg, w)
    lat.init_state(*to_comp(st), step0=0)
    for s in range(12):
        st = lattice.leapfrog_step(st)
        lat.step(1)
        errs = state_errs(lat.get_state(), st)
        assert max(errs.values()) < 1e-10, (s, errs)
    _obs_close(lat.observables(), observables.observables(st), 1e-10)


@pytest.mark.parametrize("dt,step0", [(0.5, 1), (1.0, 0), (0.25, 3)])
def test_hop_phase_and_current(dt, step0):
    """Hop schedule phase set by step0, and the deposited current against the oracle."""
    pkg = lattice_or_skip()
    w = synth.Workload("su2-16x4x4", nc=2, nz=16, nt=4, dt=dt, mu=1.0, sigma=1.5, seed=5)
    say("case: hop phase dt", dt, "step0", step0)
    p, mv = mv_setup(w)
    rA, rB = synth.mv_charges(w.seed, 2, w.nt, w.mu, w.a_T)
    st, _ = init_mv.initial_state(rA, rB, w.nz, p, mv)
    st.step = step0
    lat = new_lattice(pkg, w)
    lat.init_state(*to_comp(st), step0=step0)
    for _ in range(6):
        j = lat.deposit_current().cpu().numpy().reshape(3, 3, -1)
        if lattice.is_hop_step(st.step, p):
            _, _, jref = lattice.cpic_hop(st.U, st.rhoA, st.rhoB, p)
        else:
            jref = np.zeros_like(st.E)
        from oracle import components
        assert field_err(j, components.alg_to_comp(jref)) < 1e-12
        st = lattice.leapfrog_step(st)
        lat.step(1)
        errs = state_errs(lat.get_state(), st)
        assert max(errs.values()) < 1e-11, errs


def test_observables_and_gauss_against_oracle_on_a_generic_state():
    pkg = lattice_or_skip()
    nc, dims = 3, (6, 5, 5)
    p = lattice.Params(nc=nc, a_T=2.0, a_L=1.0, dt=0.5)
    Ua = synth.normal(101, (3,) + dims + (8,), 0.9)
    Ea = synth.normal(102, (3,) + dims + (8,), 0.4)
    st = init_mv.state_from_algebra(Ua, Ea, p)
    # a deliberate Gauss violation so the residual is non-trivial
    st.rhoA = st.rhoA * 1.001
    lat = pkg.Lattice(nc=nc, nz=dims[0], nt=dims[1], a_T=2.0, a_L=1.0, dt=0.5, fp=64)
    lat.init_state(*to_comp(st), step0=1)
    st.step = 1
    go = lat.observables()
    oo = observables.observables(st)
    _obs_close(go, oo, 1e-12)
    assert abs(go["gauss_rel"] - oo["gauss_rel"]) < 1e-10 * oo["gauss_rel"]
    assert abs(go["gauss_max"] - oo["gauss_max"]) < 1e-10 * oo["gauss_max"]
    assert go["unitarity"] < 1e-13


def test_bitwise_reproducible_rerun():
    pkg = lattice_or_skip()
    w = synth.Workload("su3-32x8x8", nc=3, nz=32, nt=8, mu=0.5, sigma=2.0, seed=120)
    rA, rB = synth.mv_charges(w.seed, 3, w.nt, w.mu, w.a_T)
    out = []
    for _ in range(2):
        lat = new_lattice(pkg, w)
        lat.init_mv(rA, rB, m_ir=w.m_ir, sigma=w.sigma)
        lat.step(17)
        out.append((lat.get_state(), lat.observables()))
    for k in ("U", "E", "rhoA", "rhoB"):
        assert np.array_equal(out[0][0][k], out[1][0][k]), k
    assert np.array_equal(out[0][1]["tmunu_z"], out[1][1]["tmunu_z"])


def test_checkpoint_resume_bitwise():
    """Run 2n steps == run n, download, upload into a new context, run n (bitwise)."""
    pkg = lattice_or_skip()
    w = synth.Workload("su2-32x6x6", nc=2, nz=32, nt=6, mu=1.0, sigma=2.0, seed=130)
    rA, rB = synth.mv_charges(w.seed, 2, w.nt, w.mu, w.a_T)
    a = new_lattice(pkg, w)
    a.init_mv(rA, rB, sigma=w.sigma)
    a.step(9)
    mid = a.get_state()
    a.step(9)
    full = a.get_state()
    b = new_lattice(pkg, w)
    b.init_state(mid["U"], mid["E"], mid["rhoA"], mid["rhoB"], step0=mid["step"])
    b.step(9)
    res = b.get_state()
    for k in ("U", "E", "rhoA", "rhoB"):
        assert np.array_equal(res[k], full[k]), k
    assert res["step"] == full["step"] == 18


def test_fp32_precision_form_against_fp64_oracle():
    """FP32 links and fields with FP64 reunitarisation every 8 steps: gauge-invariant
    observables within 1e-4 relative of the FP64 oracle."""
    pkg = lattice_or_skip()
    w = synth.Workload("su3-48x8x8", nc=3, nz=48, nt=8, mu=0.5, sigma=3.0, seed=140)
    say("case: fp32 su3 48x8x8")
    p, mv = mv_setup(w)
    rA, rB = synth.mv_charges(w.seed, 3, w.nt, w.mu, w.a_T)
    st, _ = init_mv.initial_state(rA, rB, w.nz, p, mv)
    lat = new_lattice(pkg, w, fp=32, reunit_every=8)
    lat.init_mv(rA, rB, m_ir=w.m_ir, sigma=w.sigma, zA=w.zA, zB=w.zB)
    worst = 0.0
    for blk in range(6):
        st = lattice.evolve(st, 8)
        lat.step(8)
        go, oo = lat.observables(), observables.observables(st)
        e_sl, e_H = _obs_close(go, oo, 1e-4)
        worst = max(worst, e_sl, e_H)
        assert go["unitarity"] < 1e-5
    say("fp32 worst observable error over 48 steps", worst)


def _hop_at_site(U_at, rA_at, rB_at, site, dims, p):
    """The oracle's CPIC hop (lattice.cpic_hop) evaluated on the two-layer column (z, z + 1)
    at (y, x): its layer-0 values are the hop's j_z(x) and rho_A'(x), its layer-1 value is
    rho_B'(x + z) (both rules read only U_z(x) and the charges at x and x + z).  U_at(i, pos),
    rA_at(pos), rB_at(pos) return matrices at a lattice position."""
    z, y, x = site
    nz = dims[0]
    col = [((z + k) % nz, y, x) for k in (0, 1)]
    Uc = np.stack([np.stack([U_at(i, q) for q in col]) for i in range(3)])[:, :, None, None]
    rA = np.stack([rA_at(q) for q in col])[:, None, None]
    rB = np.stack([rB_at(q) for q in col])[:, None, None]
    rA_new, rB_new, j = lattice.cpic_hop(Uc, rA, rB, p)
    return j[2, 0, 0, 0], rA_new[0, 0, 0], rB_new[1, 0, 0]


@pytest.mark.parametrize("hop", [False, True])
def test_full_size_plain_su3_sampled(hop):
    """SU(3) FP64 at the full 512 x 64 x 64 size in the benchmark's launch configuration:
    MV initial state on the GPU, then one step (the fifth, no hop, or the sixth, a hop step
    at dt = a_L/2) compared at sampled sites with the oracle: the E update of all three
    directions from the oracle's single-site force, and on the hop step the current j_z in
    E_z and both charge populations after the oracle's hop (lattice.cpic_hop) with its
    parallel transport; Gauss law and unitarity over the whole lattice."""
    pkg = lattice_or_skip()
    w = synth.PLAIN_SU3
    say("case: full-size su3 512x64x64, hop", hop)
    rA, rB = synth.mv_charges(w.seed, 3, w.nt, w.mu, w.a_T)
    lat = new_lattice(pkg, w)
    lat.init_mv(rA, rB, m_ir=w.m_ir, uv_cut=w.uv_cut, sigma=w.sigma)
    lat.step(5 if hop else 4)
    dims = (w.nz, w.nt, w.nt)
    before = from_comp(lat.get_state(), 3, dims, lattice.Params(3, w.a_T, w.a_L, w.dt))
    o = lat.observables()
    assert o["gauss_rel"] < 1e-12 and o["unitarity"] < 1e-13
    lat.step(1)
    after = lat.get_state()
    o = lat.observables()
    assert o["gauss_rel"] < 1e-12 and o["unitarity"] < 1e-13
    g = synth.rng(7)
    sites = [(int(g.integers(w.nz)), int(g.integers(w.nt)), int(g.integers(w.nt))) for _ in range(24)]
    # the nuclei (z = 128, 384) and the z seam
    sites += [(0, 0, 0), (w.nz - 1, w.nt - 1, w.nt - 1), (w.nz // 4, 5, w.nt - 1), (w.nz // 4 + 3, 9, 17),
              (3 * w.nz // 4 - 2, 40, 0), (3 * w.nz // 4, 63, 31)]
    p = before.params
    assert lattice.is_hop_step(before.step, p) == hop
    from oracle import su
    U_at = lambda i, q: before.U[i][q]
    rA_at = lambda q: before.rhoA[q]
    rB_at = lambda q: before.rhoB[q]
    rho_scale = max(np.abs(before.rhoA).max(), np.abs(before.rhoB).max())
    worst = {"E": 0.0, "rhoA": 0.0, "rhoB": 0.0}
    for (z, y, x) in sites:
        F = lattice.force_at_site(before.U, p.a, (z, y, x))
        E_ref = before.E[:, z, y, x] + p.dt * F
        if hop:
            jz, rA_new, rB_new = _hop_at_site(U_at, rA_at, rB_at, (z, y, x), dims, p)
            E_ref[2] = E_ref[2] + p.dt * jz
            s_a = (z * w.nt + y) * w.nt + x
            s_b = (((z + 1) % w.nz) * w.nt + y) * w.nt + x
            for name, got, ref in (("rhoA", after["rhoA"][:, s_a], rA_new), ("rhoB", after["rhoB"][:, s_b], rB_new)):
                e = np.abs(su.from_components(got, 3) - ref).max() / rho_scale
                worst[name] = max(worst[name], e)
                assert e < 1e-12, (name, (z, y, x), e)
        s = (z * w.nt + y) * w.nt + x
        E_got = su.from_components(after["E"][:, :, s], 3)
        e = np.abs(E_got - E_ref).max() / max(1.0, np.abs(E_ref).max())
        worst["E"] = max(worst["E"], e)
        assert e < 1e-12, ((z, y, x), e)
    say("worst sampled errors", worst)


class _SampledLinks:
    """U[i, z, y, x] read on demand from a device array in the C-ABI plain layout
    (3, r_U, V) and turned into a matrix: lets the oracle's single-site force read a
    full-size lattice without copying it to the host."""

    def __init__(self, Udev, nc, dims):
        self.U, self.nc, self.dims = Udev, nc, dims
        self.shape = (3,) + tuple(dims)
        self.cache = {}

    def __getitem__(self, key):
        i, z, y, x = key
        if key not in self.cache:
            s = (z * self.dims[1] + y) * self.dims[2] + x
            c = self.U[i, :, s].cpu().numpy()
            full = np.zeros((3, c.shape[0], 1))
            full[i, :, 0] = c
            from oracle import components
            self.cache[key] = components.comp_to_links(full, self.nc, (1, 1, 1))[i, 0, 0, 0]
        return self.cache[key]


@pytest.mark.parametrize("fp,hop", [(64, False), (32, False), (64, True), (32, True)])
def test_full_size_precision_workload_sampled(fp, hop):
    """SU(3) at the precision form's full size, 2048 x 192 x 192 (sigma = 16), FP64 and
    FP32 (reunitarisation every 8 steps): MV initial state on the GPU, Gauss law and
    unitarity over the whole lattice, and the E update of the fifth (non-hop) or sixth (hop)
    step at sampled sites recomputed by the oracle from the stored links (FP32: the stored
    FP32 values, so the bar is FP32 rounding of the update); on the hop step also the
    current in E_z and both charge populations after the oracle's hop."""
    import torch
    pkg = lattice_or_skip()
    w = synth.PRECISION_SU3
    say("case: full-size precision workload su3 2048x192x192 fp", fp, "hop", hop)
    rA, rB = synth.mv_charges(w.seed, 3, w.nt, w.mu, w.a_T)
    lat = new_lattice(pkg, w, fp=fp, reunit_every=8 if fp == 32 else 0)
    lat.init_mv(rA, rB, m_ir=w.m_ir, uv_cut=w.uv_cut, sigma=w.sigma)
    lat.step(5 if hop else 4)
    o = lat.observables()
    say("gauss_rel", o["gauss_rel"], "unitarity", o["unitarity"])
    assert o["gauss_rel"] < (1e-12 if fp == 64 else 1e-5) and o["unitarity"] < (1e-13 if fp == 64 else 1e-5)
    p = lattice.Params(3, w.a_T, w.a_L, w.dt)
    assert lattice.is_hop_step(lat.step_count, p) == hop
    f = dict(dtype=torch.float64, device=lat.device)
    U0 = torch.empty(3, lat.r, lat.V, **f)
    E0 = torch.empty(3, lat.ng, lat.V, **f)
    rA0 = torch.empty(lat.ng, lat.V, **f) if hop else None
    rB0 = torch.empty(lat.ng, lat.V, **f) if hop else None
    from paper_2009_02044_amd._lib import lib
    import ctypes as C
    vp = lambda t: C.c_void_p(t.data_ptr()) if t is not None else None
    lat._chk(lib.glasma_get_state_device(lat.ctx, vp(U0), vp(E0), vp(rA0), vp(rB0)))
    lat.step(1)
    E1 = torch.empty(3, lat.ng, lat.V, **f)
    rA1 = torch.empty(lat.ng, lat.V, **f) if hop else None
    rB1 = torch.empty(lat.ng, lat.V, **f) if hop else None
    lat._chk(lib.glasma_get_state_device(lat.ctx, None, vp(E1), vp(rA1), vp(rB1)))
    # the field scale: sites far from the nuclei carry exponentially small E whose
    # digits are rounding noise on either side (bar as max(|ref|, RMS of the field))
    rms = float(torch.sqrt(torch.mean(E1 * E1)))
    torch.cuda.synchronize()
    dims = (w.nz, w.nt, w.nt)
    Us = _SampledLinks(U0, 3, dims)
    g = synth.rng(11)
    sites = [(int(g.integers(w.nz)), int(g.integers(w.nt)), int(g.integers(w.nt))) for _ in range(16)]
    sites += [(0, 0, 0), (w.nz - 1, w.nt - 1, w.nt - 1), (w.nz // 4, 7, w.nt - 1), (3 * w.nz // 4, 0, 100)]
    from oracle import su
    worst = 0.0
    if hop:
        def charge_at(t):
            return lambda q: su.from_components(t[:, (q[0] * w.nt + q[1]) * w.nt + q[2]].cpu().numpy(), 3)
        rho_scale = max(float(rA0.abs().max()), float(rB0.abs().max()))
        sites += [(w.nz // 4 + 5, 3, 3), (3 * w.nz // 4 - 6, 150, 191)]   # inside the nuclei
    for (z, y, x) in sites:
        s = (z * w.nt + y) * w.nt + x
        F = lattice.force_at_site(Us, p.a, (z, y, x))
        E_ref = su.from_components(E0[:, :, s].cpu().numpy(), 3) + p.dt * F
        if hop:
            jz, rA_new, rB_new = _hop_at_site(lambda i, q: Us[(i,) + tuple(q)], charge_at(rA0), charge_at(rB0),
                                              (z, y, x), dims, p)
            E_ref[2] = E_ref[2] + p.dt * jz
            s_b = (((z + 1) % w.nz) * w.nt + y) * w.nt + x
            for name, t, sg, ref in (("rhoA", rA1, s, rA_new), ("rhoB", rB1, s_b, rB_new)):
                e = np.abs(su.from_components(t[:, sg].cpu().numpy(), 3) - ref).max() / rho_scale
                assert e < (1e-12 if fp == 64 else 1e-6), (name, (z, y, x), e)
        E_got = su.from_components(E1[:, :, s].cpu().numpy(), 3)
        scale = max(np.abs(E_ref).max(), rms)
        err = np.abs(E_got - E_ref).max() / scale
        worst = max(worst, err)
        # FP32: the force sums ~100 products of O(1) link entries in FP32 (unit roundoff
        # 6e-8) while E is small on most of the lattice (RMS ~ 1/4 of the peak)
        assert err < (1e-10 if fp == 64 else 5e-5), ((z, y, x), err)
    say("worst sampled E-update error (relative to max(|E|, RMS E))", worst)


@pytest.mark.parametrize("nc,nz,nt", [(3, 3, 64), (3, 4, 32), (2, 4, 16), (3, 4, 12), (3, 2, 2), (2, 2, 3),
                                      (3, 5, 2), (3, 2, 65)])
def test_leapfrog_generic_state_row_layouts(nc, nz, nt):
    """Per-component parity on a generic state (random links and fields, charges from the
    Gauss law) for rows of 64, 32 and 16 sites (a wavefront holds whole rows: x neighbours
    come from adjacent lanes, backward -x plaquettes from the neighbour lane) and of 12
    sites (rows cross wavefronts: every neighbour from memory); the smallest lattices (two
    sites per row: x + 1 and x - 1 are the same site; nz = 2: z + 1 = z - 1) and a row of
    65 (one lane past a wavefront); steps 1..6 include hops."""
    pkg = lattice_or_skip()
    say(f"case: generic state su{nc} {nz}x{nt}x{nt}")
    dims = (nz, nt, nt)
    ng = nc * nc - 1
    p = lattice.Params(nc=nc, a_T=4.0, a_L=1.0, dt=0.5)
    Ua = synth.normal(200 + nt, (3,) + dims + (ng,), 0.6)
    Ea = synth.normal(300 + nt, (3,) + dims + (ng,), 0.3)
    st = init_mv.state_from_algebra(Ua, Ea, p)
    lat = pkg.Lattice(nc=nc, nz=nz, nt=nt, a_T=4.0, a_L=1.0, dt=0.5, fp=64)
    lat.init_state(*to_comp(st), step0=0)
    for s in range(6):
        st = lattice.leapfrog_step(st)
        lat.step(1)
        errs = state_errs(lat.get_state(), st)
        assert max(errs.values()) < 1e-10, (s, errs)
    go, oo = lat.observables(), observables.observables(st)
    _obs_close(go, oo, 1e-10)
    assert go["gauss_rel"] < 1e-12


def test_rest_frame_against_oracle():
    """Local rest frame per layer (glasma_rest_frame on the observe slices) against the
    oracle's eps_loc and frame velocity from its own slices, two colliding nuclei mid-way
    through their overlap."""
    pkg = lattice_or_skip()
    import torch
    w = synth.Workload("su2-64x8x8", nc=2, nz=64, nt=8, mu=1.0, sigma=4.0, seed=1001)
    say("case: rest frame su2 64x8x8")
    p, mv = mv_setup(w)
    rA, rB = synth.mv_charges(w.seed, w.nc, w.nt, w.mu, w.a_T)
    st, _ = init_mv.initial_state(rA, rB, w.nz, p, mv)
    lat = new_lattice(pkg, w)
    lat.init_state(*to_comp(st), step0=0)
    n = 30
    st = lattice.evolve(st, n)
    lat.step(n)
    obs = lat.obs_buffer()
    lat.observe(obs)
    got = lat.rest_frame(obs)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    el, v = observables.local_rest_frame(observables.tmunu_slices(st)[0])
    scale = np.abs(observables.tmunu_slices(st)[0][0]).max()
    assert np.max(np.abs(got[0] - el)) < 1e-8 * scale, np.max(np.abs(got[0] - el)) / scale
    big = np.abs(el) > 1e-3 * scale
    assert np.max(np.abs(got[1] - v)[big]) < 1e-6
    assert np.all(np.abs(got[1]) < 1.0)


@pytest.mark.parametrize("n", [5, 6])
@pytest.mark.parametrize("nc,nz,nt,fp", [(3, 4, 64, 64), (2, 4, 64, 64), (3, 2, 128, 64), (3, 6, 8, 64),
                                         (3, 5, 12, 64), (2, 4, 12, 64), (3, 4, 64, 32), (3, 3, 12, 32),
                                         (2, 4, 8, 32)])
def test_step_observe_equals_step_then_observe(nc, nz, nt, fp, n):
    """glasma_step_observe(n) against glasma_step(n - 1), glasma_observe, glasma_step(1):
    the same observables and the same final state.  The FP64 cases with nt a multiple of 64
    take the fused observing step (Gauss pass plus energy slots inside the step kernel, x
    neighbours from adjacent lanes at nt = 64 and from memory at nt = 128); the others the
    passes around a plain step (x neighbours from adjacent lanes at nt = 8 and 64, from memory
    at nt = 12), whose E(t + dt/2) is the step's own (in FP32 its FP32 update, where the
    standalone pass recomputes it in double).  The observing step is a step without a hop for
    n = 5 and one with a hop for n = 6 (hops on odd step indices)."""
    pkg = lattice_or_skip()
    import torch
    say(f"case: step_observe su{nc} {nz}x{nt}x{nt} fp{fp} n={n}")
    dims = (nz, nt, nt)
    ng = nc * nc - 1
    p = lattice.Params(nc=nc, a_T=4.0, a_L=1.0, dt=0.5)
    st = init_mv.state_from_algebra(synth.normal(400 + nt, (3,) + dims + (ng,), 0.6),
                                    synth.normal(500 + nt, (3,) + dims + (ng,), 0.3), p)
    st.rhoA = st.rhoA * 1.001          # a non-trivial Gauss residual
    comp = to_comp(st)
    a = pkg.Lattice(nc=nc, nz=nz, nt=nt, a_T=4.0, a_L=1.0, dt=0.5, fp=fp)
    b = pkg.Lattice(nc=nc, nz=nz, nt=nt, a_T=4.0, a_L=1.0, dt=0.5, fp=fp)
    a.init_state(*comp, step0=0)
    b.init_state(*comp, step0=0)
    oa, ob = a.obs_buffer(), b.obs_buffer()
    assert lattice.is_hop_step(n - 1, p) == (n == 6)
    a.step_observe(n, oa)
    b.step(n - 1)
    b.observe(ob)
    b.step(1)
    torch.cuda.synchronize()
    ga, gb = pkg.Lattice.unpack_obs(oa, nz), pkg.Lattice.unpack_obs(ob, nz)
    sc = np.abs(gb["tmunu_z"]).max(axis=1, keepdims=True)
    tol = 1e-11 if fp == 64 else 1e-5
    assert np.max(np.abs(ga["tmunu_z"] - gb["tmunu_z"]) / sc) < tol
    assert abs(ga["energy"] - gb["energy"]) < tol * abs(gb["energy"])
    for k in ("gauss_l2", "rho_l2", "gauss_max"):
        if k in gb:
            assert abs(ga[k] - gb[k]) <= 1e-9 * abs(gb[k]) + 1e-14, (k, ga[k], gb[k])
    assert abs(ga["unitarity"] - gb["unitarity"]) < 1e-12 + 1e-6 * (fp == 32)
    assert ga["nonfinite"] == 0 and gb["nonfinite"] == 0
    sa, sb = a.get_state(), b.get_state()
    for k in ("U", "E", "rhoA", "rhoB"):
        assert np.array_equal(sa[k], sb[k]), k


@pytest.mark.parametrize("nc,fp", [(3, 64), (2, 64), (3, 32)])
def test_gauge_invariance_of_the_gpu_evolution(nc, fp):
    """A random gauge transformation of the initial state (links, E and charges) leaves the
    GPU's T^{mu nu} slices, H and Gauss residual unchanged, at the start and after 6 steps
    through charge hops: the update and the CPIC hop are gauge covariant on the GPU too."""
    pkg = lattice_or_skip()
    nz, nt = 8, 16
    say(f"case: gauge invariance su{nc} {nz}x{nt}x{nt} fp{fp}")
    dims = (nz, nt, nt)
    ng = nc * nc - 1
    p = lattice.Params(nc=nc, a_T=4.0, a_L=1.0, dt=0.5)
    st = init_mv.state_from_algebra(synth.normal(71, (3,) + dims + (ng,), 0.5),
                                    synth.normal(72, (3,) + dims + (ng,), 0.3), p)
    from oracle import su
    Omega = su.expi(su.from_components(synth.normal(73, dims + (ng,), 1.5), nc))
    st2 = lattice.gauge_transform(st, Omega)
    lats = []
    for s_ in (st, st2):
        lat = pkg.Lattice(nc=nc, nz=nz, nt=nt, a_T=4.0, a_L=1.0, dt=0.5, fp=fp)
        lat.init_state(*to_comp(s_), step0=0)
        lats.append(lat)
    tol = 1e-11 if fp == 64 else 2e-5
    for n in (0, 6):
        if n:
            for lat in lats:
                lat.step(n)
        o1, o2 = lats[0].observables(), lats[1].observables()
        scale = np.abs(o1["tmunu_z"]).max(axis=1, keepdims=True)
        err = np.max(np.abs(o1["tmunu_z"] - o2["tmunu_z"]) / scale)
        err_H = abs(o1["energy"] - o2["energy"]) / abs(o1["energy"])
        say(f"  after {n} steps: slices {err:.1e}, H {err_H:.1e}, gauss {o1['gauss_rel']:.1e} {o2['gauss_rel']:.1e}")
        assert err < tol and err_H < tol
        assert o2["gauss_rel"] < (1e-12 if fp == 64 else 1e-5)


def test_energy_conservation_in_free_evolution():
    """No charges, E = 0 and random links (the Gauss law holds with rho = 0): the leapfrog
    keeps H within bounded oscillations that shrink with dt (symplectic update; a random-link
    state has much of its energy in lattice-scale modes, so the oscillation is large at
    dt = a_L/2), with no drift, over 200 a_L of time on the GPU; the Gauss residual stays
    at round-off."""
    pkg = lattice_or_skip()
    nc, nz, nt = 3, 16, 16
    say(f"case: free evolution su{nc} {nz}x{nt}x{nt}, t = 200")
    dims = (nz, nt, nt)
    p = lattice.Params(nc=nc, a_T=4.0, a_L=1.0, dt=0.5)
    st = init_mv.state_from_algebra(synth.normal(81, (3,) + dims + (8,), 0.12), np.zeros((3,) + dims + (8,)), p)
    assert np.abs(st.rhoA).max() == 0 and np.abs(st.rhoB).max() == 0
    fl, dr = {}, {}
    for dt in (0.5, 0.25):
        lat = pkg.Lattice(nc=nc, nz=nz, nt=nt, a_T=4.0, a_L=1.0, dt=dt, fp=64)
        lat.init_state(*to_comp(st), step0=0)
        per = int(round(10 / dt))
        H, G = [], []
        for k in range(21):
            if k:
                lat.step(per)
            o = lat.observables()
            H.append(o["energy"])
            G.append(o["gauss_max"])     # absolute: rho = 0
        H = np.array(H)
        fl[dt] = np.abs(H - H[0]).max() / H[0]
        dr[dt] = abs(H[11:].mean() - H[1:11].mean()) / H[0]
        say(f"  dt {dt}: max |H - H0| / H0 {fl[dt]:.3e}, drift between halves {dr[dt]:.1e}, max |G| {max(G):.1e}")
        assert max(G) < 1e-11
    # the oscillation shrinks with dt (the dt^2 law itself is pinned on the oracle; here the
    # start E(-dt/2) = 0 differs between the two runs) and does not drift
    assert fl[0.25] < 0.6 * fl[0.5]
    assert dr[0.5] < 0.1 * fl[0.5] and dr[0.25] < 0.1 * fl[0.25]


@pytest.mark.parametrize("nt,k", [(8, (0, 1, 2)), (8, (0, 3, 1)), (12, (0, 2, 3))])
def test_dispersion_relation_of_small_plane_waves(nt, k):
    """A small single-colour plane wave A_x ~ cos(k.x) on the GPU: its linearised leapfrog
    evolution obeys A(t+dt) + A(t-dt) = 2 cos(w dt) A(t) with the lattice dispersion
    (2/dt)^2 sin^2(w dt/2) = sum_i (2/a_i)^2 sin^2(k_i a_i/2) (closed form; rows of 8 sites
    take the lane-exchange path, rows of 12 the memory path)."""
    pkg = lattice_or_skip()
    from oracle import su
    nc, nz, a_T, dt = 2, 16, 4.0, 0.5
    say(f"case: dispersion nt {nt} k {k}")
    dims = (nz, nt, nt)
    a = (a_T, a_T, 1.0)
    p = lattice.Params(nc=nc, a_T=a_T, a_L=1.0, dt=dt)
    nx = np.arange(nt)[None, None, :]
    ny = np.arange(nt)[None, :, None]
    nzv = np.arange(nz)[:, None, None]
    kv = [2 * np.pi * k[0] / nt, 2 * np.pi * k[1] / nt, 2 * np.pi * k[2] / nz]
    phase = kv[0] * nx + kv[1] * ny + kv[2] * nzv
    alg = np.zeros((3,) + dims + (3,))
    alg[0, ..., 2] = a[0] * 1e-6 * np.cos(phase)        # polarisation x, k has no x part
    z = np.zeros(dims + (2, 2), complex)
    st = lattice.State(su.expi(su.from_components(alg, nc)), np.zeros((3,) + dims + (2, 2), complex), z, z.copy(), 0, p)
    lat = pkg.Lattice(nc=nc, nz=nz, nt=nt, a_T=a_T, a_L=1.0, dt=dt, fp=64)
    lat.init_state(*to_comp(st), step0=0)
    A = []
    for _ in range(4):
        g = from_comp(lat.get_state(), nc, dims, p)
        A.append(su.to_components(su.logi(g.U[0]))[..., 2])
        lat.step(1)
    A = np.array(A)
    msk = np.abs(A[1]) > 0.3 * np.abs(A[1]).max()
    cos_w = ((A[2] + A[0]) / (2 * A[1]))[msk]
    Om2 = sum((2 / a[i]) ** 2 * np.sin(kv[i] / 2) ** 2 for i in range(3))
    expect = 1 - dt ** 2 * Om2 / 2
    say("  cos(w dt)", float(np.mean(cos_w)), "closed form", expect, "max dev", float(np.abs(cos_w - expect).max()))
    np.testing.assert_allclose(cos_w, expect, rtol=1e-8, atol=1e-9)


@pytest.mark.parametrize("nc,fp,nt", [(2, 64, 16), (2, 32, 21), (3, 64, 21), (3, 32, 16), (3, 64, 64), (3, 32, 2)])
def test_link_and_site_steps_agree(nc, fp, nt):
    """Small lattices take a step with a thread per link, larger ones with a thread per site: nz
    layers against the same layers repeated along z until the other kernel runs.  Same
    operations in the same order: bitwise equal, through hops, no-hop steps and (FP32)
    reunitarising steps, with rows in wavefronts (2, 16, 64) and across them (21)."""
    pkg = lattice_or_skip()
    nz = 4
    reps = 90000 // (nz * nt * nt) + 1
    w = synth.Workload(f"su{nc}-{nz}x{nt}", nc=nc, nz=nz, nt=nt, mu=0.5, sigma=0.8, seed=430 + nt)
    print("case: link and site steps", w.name, "fp", fp, "x", reps, flush=True)
    p, mv = mv_setup(w)
    rA, rB = synth.mv_charges(w.seed, nc, nt, w.mu, w.a_T)
    st, _ = init_mv.initial_state(rA, rB, nz, p, mv)
    arrs = to_comp(st)
    V = nz * nt * nt
    kw = dict(nc=nc, nt=nt, a_T=w.a_T, a_L=w.a_L, dt=w.dt, fp=fp, reunit_every=4 if fp == 32 else 0)
    one, many = pkg.Lattice(nz=nz, **kw), pkg.Lattice(nz=nz * reps, **kw)
    one.init_state(*arrs, step0=0)
    many.init_state(*[np.tile(x, reps) for x in arrs], step0=0)
    one.step(6)
    many.step(6)
    a, b = one.get_state(), many.get_state()
    for k in ("U", "E", "rhoA", "rhoB"):
        x = b[k].reshape(*b[k].shape[:-1], reps, V)
        assert np.array_equal(x, np.broadcast_to(a[k][..., None, :], x.shape)), k


@pytest.mark.parametrize("nc,nz,nt", [(2, 9, 100), (3, 5, 100), (2, 6, 128)])
def test_step_of_layers_in_bands(nc, nz, nt):
    """Layers of more than 9216 sites are swept in bands (the last one narrower at nt = 100): two
    steps against the oracle; an observing step between them (fused at nt = 128)."""
    pkg = lattice_or_skip()
    w = synth.Workload(f"su{nc}-{nz}x{nt}", nc=nc, nz=nz, nt=nt, mu=0.5, sigma=1.0, seed=440 + nt)
    say("case: layers in bands", w.name)
    p, mv = mv_setup(w)
    rA, rB = synth.mv_charges(w.seed, nc, nt, w.mu, w.a_T)
    st, _ = init_mv.initial_state(rA, rB, nz, p, mv)
    lat = new_lattice(pkg, w)
    lat.init_state(*to_comp(st), step0=0)
    buf = lat.obs_buffer()
    lat.step_observe(2, buf)
    st = lattice.leapfrog_step(st)
    _obs_close(pkg.Lattice.unpack_obs(buf, nz), observables.observables(st), 1e-8)
    st = lattice.leapfrog_step(st)
    errs = state_errs(lat.get_state(), st)
    assert max(errs.values()) < 1e-10, errs


@pytest.mark.parametrize("nz,nt", [(129, 49), (129, 48), (128, 49), (5, 49), (2, 200)])
def test_observables_over_partial_sums(nz, nt):
    """The observables' partial sums: 10 of a layer added up beforehand (129 x 49), 9 by a lane
    (129 x 48), over 2 lanes, over 16 and over 64: slices and scalars against the oracle."""
    pkg = lattice_or_skip()
    say("case: partial sums", nz, nt)
    p = lattice.Params(nc=2, a_T=4.0, a_L=1.0, dt=0.5)
    st = init_mv.state_from_algebra(synth.normal(600 + nt, (3, nz, nt, nt, 3), 0.6),
                                    synth.normal(700 + nt, (3, nz, nt, nt, 3), 0.3), p)
    lat = pkg.Lattice(nc=2, nz=nz, nt=nt, a_T=4.0, a_L=1.0, dt=0.5, fp=64)
    lat.init_state(*to_comp(st), step0=0)
    go, oo = lat.observables(), observables.observables(st)
    _obs_close(go, oo, 1e-11)
    for k in ("gauss_l2", "rho_l2", "gauss_max"):
        if k in oo:
            assert abs(go[k] - oo[k]) <= 1e-11 * abs(oo[k]) + 1e-14, k


@pytest.mark.parametrize("nc,nz,nt", [(2, 129, 49), (2, 129, 48), (2, 128, 49), (2, 5, 49), (2, 2, 200), (3, 33, 33)])
def test_residual_sums_over_partial_sums(nc, nz, nt):
    """The sums over all layers, ||G||_2 and ||rho||_2, and max |G| at the same numbers of partial
    sums, of a state off the Gauss law (where they are not rounding alone).  A site's G is some 60
    roundings off, each partial sum and the sum over them no more than 40: 1e-12 leaves 40x."""
    pkg = lattice_or_skip()
    say("case: residual sums", nc, nz, nt)
    p = lattice.Params(nc=nc, a_T=4.0, a_L=1.0, dt=0.5)
    ng = nc * nc - 1
    st = init_mv.state_from_algebra(synth.normal(800 + nt, (3, nz, nt, nt, ng), 0.6),
                                    synth.normal(810 + nt, (3, nz, nt, nt, ng), 0.3), p)
    st.E += su.from_components(synth.normal(820 + nt, (3, nz, nt, nt, ng), 0.3), nc)
    lat = pkg.Lattice(nc=nc, nz=nz, nt=nt, a_T=4.0, a_L=1.0, dt=0.5, fp=64)
    lat.init_state(*to_comp(st), step0=0)
    buf = lat.obs_buffer()
    lat.observe(buf)
    o = pkg.Lattice.unpack_obs(buf, nz)
    rel, gmax = lattice.gauss_residual(st)
    rho = np.sqrt(np.sum(su.algebra_norm2(st.rhoA + st.rhoB)))
    for k, ref in (("gauss_l2", rel * rho), ("rho_l2", rho), ("gauss_rel", rel), ("gauss_max", gmax)):
        assert abs(o[k] - ref) <= 1e-12 * ref, (k, o[k], ref)
    assert rel > 0.1


def _tiled_pair(pkg, nc, fp, nz, nt, reps, seed):
    """A lattice of nz layers and one of the same layers repeated `reps` times along z."""
    w = synth.Workload(f"su{nc}-{nz}x{nt}", nc=nc, nz=nz, nt=nt, mu=0.5, sigma=0.8, seed=seed)
    print("case:", w.name, "fp", fp, "x", reps, flush=True)
    p, mv = mv_setup(w)
    rA, rB = synth.mv_charges(w.seed, nc, nt, w.mu, w.a_T)
    st, _ = init_mv.initial_state(rA, rB, nz, p, mv)
    arrs = to_comp(st)
    kw = dict(nc=nc, nt=nt, a_T=w.a_T, a_L=w.a_L, dt=w.dt, fp=fp, reunit_every=4 if fp == 32 else 0)
    one, many = pkg.Lattice(nz=nz, **kw), pkg.Lattice(nz=nz * reps, **kw)
    one.init_state(*arrs, step0=0)
    many.init_state(*[np.tile(x, reps) for x in arrs], step0=0)
    return one, many


def _same_layers(one, many, reps):
    a, b = one.get_state(), many.get_state()
    for k in ("U", "E", "rhoA", "rhoB"):
        x = b[k].reshape(*b[k].shape[:-1], reps, one.V)
        assert np.array_equal(x, np.broadcast_to(a[k][..., None, :], x.shape)), k


@pytest.mark.parametrize("nc,fp,nt", [(3, 64, 150), (2, 64, 150), (3, 32, 150), (2, 32, 192), (3, 64, 128), (2, 64, 192)])
def test_bands_of_several_layers(nc, fp, nt):
    """Large layers in bands with two and three layers per XCD (the last band narrower at nt = 150:
    work-groups in 30, 30, 28) against three layers, one per XCD, which need no order: steps
    with and without a hop and an observing step (fused for FP64 at nt = 128, 192): the state
    bitwise; a layer's partial sums, n = nt^2 / 256 of them, are added in another order (over more
    lanes for fewer layers), so the slices agree to 2 n roundings of the layer's energy density,
    which bounds the terms of every slice."""
    pkg = lattice_or_skip()
    nz, reps = 3, 6
    one, many = _tiled_pair(pkg, nc, fp, nz, nt, reps, 450 + nt)
    for lat in (one, many):
        lat.buf = lat.obs_buffer()
        lat.step_observe(4, lat.buf)
    a = pkg.Lattice.unpack_obs(one.buf, nz)["tmunu_z"]
    b = pkg.Lattice.unpack_obs(many.buf, nz * reps)["tmunu_z"]
    assert np.all(np.abs(b - np.tile(a, reps)) <= (nt * nt // 256 + 1) * 2.0 ** -52 * np.tile(a[0], reps))
    _same_layers(one, many, reps)


@pytest.mark.parametrize("nc,fp,nz,nt,sites", [(2, 64, 4, 16, 300000), (2, 32, 4, 21, 300000), (3, 64, 3, 8, 100000),
                                               (3, 32, 4, 16, 200000), (3, 64, 5, 21, 100000), (2, 32, 2, 48, 200000),
                                               (3, 64, 2, 48, 39168), (3, 32, 3, 9, 120000)])
def test_link_step_at_its_limits(nc, fp, nz, nt, sites):
    """A step by links (few layers) against a step by sites (the same layers repeated until more waves
    per XCD than any limit of the rule): both kinds of rows, layers of one wave (8), sizes that
    the number of sites alone does not decide (39 168 sites in 17 layers); bitwise, hops and no-hop
    steps, FP32 with reunitarising steps."""
    pkg = lattice_or_skip()
    reps = sites // (nz * nt * nt) + 1
    one, many = _tiled_pair(pkg, nc, fp, nz, nt, reps, 470 + nt)
    one.step(6)
    many.step(6)
    _same_layers(one, many, reps)
