"""Finite electronic temperature on the GPU: the Fermi operator by the
recursive expansion (rocBLAS GEMMs, Newton-Schulz inverses, canonical mu by
Newton) against the oracle's recursion at the same number of steps and against
the definition by eigendecomposition."""
import sys
import time

import numpy as np
import pytest

import synth
from oracle import fermi, observables, sp2 as osp2, tb as otb

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    import torch
    import paper_1203_6836_amd as p
    c = p.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def to_dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def lattice(dims, seed):
    w = synth.small_workload(dims, seed)
    return w, otb.hamiltonian(w.positions(), None, synth.STATIC_MODEL)


@pytest.mark.parametrize("dims,seed,kT,n", [((3, 3, 3), 1, 0.5, 10), ((3, 3, 3), 2, 0.5, 14),
                                            ((4, 4, 9), 3, 1.0, 12)])
def test_fixed_mu_matches_oracle_recursion(ctx, dims, seed, kT, n):
    w, H = lattice(dims, seed)
    say(f"case fermi fixed mu N={w.n_orb} kT={kT} n={n}")
    e = np.linalg.eigvalsh(H)
    mu = 0.5 * (e[w.n_occ - 1] + e[w.n_occ])
    ref = fermi.recursive_fermi(H, mu, kT, n)
    D, mu_out, passes = ctx.sp2_fermi_density_matrix(to_dev(H), w.n_occ, kT, n, mu=mu, max_newton=0)
    D = D.cpu().numpy()
    err = float(np.abs(D - ref).max())
    say(f"  max|D - oracle| {err:.2e}, passes {passes}")
    assert passes == 1 and mu_out == mu
    assert np.array_equal(D, D.T)
    assert err < 1e-10


@pytest.mark.parametrize("dims,seed,kT", [((3, 3, 3), 1, 0.5), ((4, 4, 8), 5, 0.25), ((4, 4, 9), 3, 2.0)])
def test_canonical_matches_oracle_and_definition(ctx, dims, seed, kT):
    w, H = lattice(dims, seed)
    say(f"case fermi canonical N={w.n_orb} kT={kT}")
    X, mu_ref, its_ref = fermi.recursive_fermi_canonical(H, w.n_occ, kT, 16, tol=1e-9)
    Dd, mu_def, _ = fermi.fermi_density(H, w.n_occ, kT)
    D, mu, passes = ctx.sp2_fermi_density_matrix(to_dev(H), w.n_occ, kT, 16, tol=1e-9)
    D = D.cpu().numpy()
    e_rec = float(np.abs(D - X).max())
    e_def = float(np.abs(D - Dd).max())
    say(f"  passes gpu={passes} oracle={its_ref}, mu {mu:.12f} (oracle {mu_ref:.12f}, definition {mu_def:.12f}), "
        f"max|D - recursion| {e_rec:.2e}, max|D - definition| {e_def:.2e}, Tr D - n_occ {np.trace(D) - w.n_occ:+.1e}")
    assert abs(passes - its_ref) <= 1
    assert abs(mu - mu_ref) < 1e-9 and abs(mu - mu_def) < 1e-8
    assert abs(np.trace(D) - w.n_occ) < 1e-9
    assert e_rec < 1e-9 and e_def < 1e-8


def test_low_temperature_limit_is_the_projector(ctx):
    """kT = 0.02 eV on the gapped wire (gap ~5 eV): D equals the zero-temperature
    projector (the oracle's SP2 result) to the Fermi tail's e^(-gap/2kT)."""
    w = synth.gapped_workload(2)
    H = otb.hamiltonian(w.positions(), None, synth.GAPPED_MODEL)
    say(f"case fermi low T N={w.n_orb}")
    P = osp2.sp2(H, w.n_occ).D
    D, mu, passes = ctx.sp2_fermi_density_matrix(to_dev(H), w.n_occ, 0.02, 20, tol=1e-9)
    D = D.cpu().numpy()
    err = float(np.abs(D - P).max())
    say(f"  mu {mu:.6f}, passes {passes}, max|D - projector| {err:.2e}")
    assert err < 1e-9


def test_fermi_rejects_bad_arguments(ctx):
    import paper_1203_6836_amd as p
    w, H = lattice((2, 2, 2), 1)
    Hd = to_dev(H)
    say("case fermi argument checks")
    for kw in ({"kT": 0.0, "n_steps": 12}, {"kT": 0.5, "n_steps": 0}, {"kT": 0.5, "n_steps": 2},
               {"kT": 0.5, "n_steps": 12, "max_newton": 0}):
        with pytest.raises(p.Sp2Error) as ei:
            ctx.sp2_fermi_density_matrix(Hd, w.n_occ, **kw)
        assert ei.value.status == p.SP2_EINVAL, kw
    Hb = H.copy()
    Hb[0, 1] += 1.0
    with pytest.raises(p.Sp2Error) as ei:
        ctx.sp2_fermi_density_matrix(to_dev(Hb), w.n_occ, 0.5, 12)
    assert ei.value.status == p.SP2_EINVAL
    e_lo = osp2.gershgorin(H)[0]
    with pytest.raises(p.Sp2Error) as ei:   # one pass from a mu near the bottom of the spectrum
        ctx.sp2_fermi_density_matrix(Hd, w.n_occ, 0.5, 12, mu=e_lo + 1.0, max_newton=1)
    assert ei.value.status == p.SP2_ENOCONV


def test_fermi_full_size_against_definition(ctx):
    """N = 2048 (512 atoms): the canonical Fermi operator at kT = 0.5 eV with 16
    steps against the definition (eigendecomposition on the host), and its
    GEMM rate."""
    import torch
    w, H = lattice((8, 8, 8), 7)
    say(f"case fermi N={w.n_orb}")
    Hd = to_dev(H)
    ctx.sp2_fermi_density_matrix(Hd, w.n_occ, 0.5, 16, tol=1e-8)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    D, mu, passes = ctx.sp2_fermi_density_matrix(Hd, w.n_occ, 0.5, 16, tol=1e-8)
    torch.cuda.synchronize()
    s = time.perf_counter() - t0
    prods = ctx.last_fermi_products
    assert passes * 2 * 16 <= prods <= passes * 10 * 16
    tf = prods * 2.0 * w.n_orb ** 3 / s / 1e12
    Dd, mu_def, _ = fermi.fermi_density(H, w.n_occ, 0.5, solver="lapack")   # Jacobi is too slow at N = 2048
    err = float(np.abs(D.cpu().numpy() - Dd).max())
    say(f"  {s * 1e3:.1f} ms, {passes} passes, {prods} products, {tf:.1f} TF/s in GEMMs, mu - mu_def {mu - mu_def:+.1e}, "
        f"max|D - definition| {err:.2e}")
    assert err < 1e-7 and abs(mu - mu_def) < 1e-6


def test_finite_temperature_forces_match_oracle(ctx):
    """Forces and U at constant n with the Fermi D (kT = 0.5 eV): the GPU's
    Fermi operator fed to the GPU's force kernel against the oracle's
    definition and force expression (-dA/dR, A = U - T_e S, by the oracle's
    finite-difference pin)."""
    m = synth.MD_MODEL
    dims = (3, 3, 3)
    pos = synth.lattice_positions(dims, seed=21)
    nat = len(pos)
    n = np.random.default_rng(5).uniform(-0.2, 0.2, nat)
    n_occ = 2 * nat
    say(f"case fermi forces N={4 * nat} kT=0.5")
    A, Dd, mu_d = fermi.free_energy(pos, n, m, n_occ, 0.5)
    F_ref = observables.forces(pos, n, Dd, m)
    U_ref = observables.potential_energy(pos, n, Dd, m)
    xyz, nd = to_dev(pos), to_dev(n)
    H = ctx.tb_hamiltonian(m, xyz, nd)
    D, mu, _ = ctx.sp2_fermi_density_matrix(H, n_occ, 0.5, 16, tol=1e-9)
    q = ctx.sp2_mulliken(D, nat)
    F, U = ctx.tb_forces(m, xyz, D, q, nd)
    dF = float(np.abs(F.cpu().numpy() - F_ref).max())
    say(f"  mu {mu:.10f} (definition {mu_d:.10f}), max|dF| {dF:.2e} (max|F| {np.abs(F_ref).max():.1f}), "
        f"dU {U - U_ref:+.2e}")
    assert abs(mu - mu_d) < 1e-8
    assert dF < 1e-8 and abs(U - U_ref) < 1e-8


@pytest.mark.parametrize("dims,seed,kT", [((3, 3, 3), 1, 0.5), ((4, 4, 8), 5, 0.25), ((4, 4, 9), 3, 2.0)])
def test_entropy_matches_definition(ctx, dims, seed, kT):
    """S / k_B by Chebyshev moments on the GPU against the oracle's entropy of
    the eigenvalue occupations at the same mu."""
    import paper_1203_6836_amd as p
    w, H = lattice(dims, seed)
    say(f"case fermi entropy N={w.n_orb} kT={kT}")
    e = np.linalg.eigvalsh(H)
    mu = fermi.canonical_mu(e, w.n_occ, 1.0 / kT)
    S_ref = fermi.entropy(fermi.fermi_occupations(e, mu, 1.0 / kT))
    S, m = ctx.sp2_fermi_entropy(to_dev(H), mu, kT)
    say(f"  S {S:.12f} (oracle {S_ref:.12f}), rel {(S - S_ref) / S_ref:+.1e}, {m} coefficients")
    assert abs(S - S_ref) < 1e-10 * S_ref
    with pytest.raises(p.Sp2Error) as ei:
        ctx.sp2_fermi_entropy(to_dev(H), mu, 0.01)
    assert ei.value.status == p.SP2_EINVAL


def test_finite_temperature_xlbomd_matches_oracle(ctx):
    """XL-BOMD at kT = 0.5 eV (Fermi operator, its entropy in the free energy,
    forces of the Fermi D every step) on the 3 x 3 x 3 cluster, whose gap
    (0.16 eV) is well below kT: 20 steps from self-consistent finite-T charges
    against the oracle integrator with the Fermi operator by definition."""
    import paper_1203_6836_amd as p
    from oracle import xlbomd as oxl
    say("case fermi xlbomd 3x3x3 20 steps kT=0.5")
    m = synth.MD_MODEL
    pos = synth.lattice_positions((3, 3, 3), seed=21)
    nat, nocc = len(pos), 2 * len(pos)
    vel = synth.maxwell_velocities(nat, 300.0, m.mass, seed=5)
    n0 = np.zeros(nat)
    for _ in range(2000):   # finite-T SCF by linear mixing
        q = oxl.evaluate(pos, n0, m, nocc, want_forces=False, kT=0.5)["q"]
        if np.abs(q - n0).max() < 1e-11:
            break
        n0 = n0 + 0.1 * (q - n0)
    assert np.abs(q - n0).max() < 1e-11
    opts = oxl.XLOptions(kT=0.5, kappa=p.KAPPA_FINITE_T)   # the kappa rescaling of finite-T runs
    assert p.KAPPA_FINITE_T == 0.75 * oxl.K5_KAPPA
    ost, olog = oxl.run(oxl.init_state(pos, vel, m, nocc, opts, n0), m, nocc, opts, 20)
    md = ctx.xlbomd_create(m, pos, vel, n0, dt_fs=opts.dt_fs, kappa=opts.kappa, alpha=opts.alpha,
                           c=opts.c, sp2_opts=p.options("fp64"), kT=0.5, fermi_steps=16)
    glog = md.xlbomd_run(20)
    xyz, v, q, n = md.xlbomd_get()
    md.close()
    dx = float(np.abs(xyz - ost.pos).max())
    eg = np.array([r["etot"] for r in glog])
    eo = np.array([r["etot"] for r in olog])
    passes = [r["sp2_iterations"] for r in glog]
    say(f"  max|dx| {dx:.1e} A, max|dE_tot| {np.abs(eg - eo).max():.1e} eV, E_tot spread {np.ptp(eo) / nat:.1e} "
        f"eV/atom, Newton passes per step {passes[:3]}..{passes[-3:]}")
    np.testing.assert_allclose(xyz, ost.pos, atol=1e-9)
    np.testing.assert_allclose(v, ost.vel, atol=1e-9)
    # the step's canonical mu is solved to |Tr D - n_occ| < 1e-9, which bounds
    # how closely the charges, and the auxiliary charges built from them, agree
    np.testing.assert_allclose(n, ost.hist[0], atol=2e-8)
    assert np.abs(eg - eo).max() < 1e-7


def test_finite_temperature_checkpoint_resume_is_bit_identical(ctx):
    """A checkpoint of a kT > 0 integrator carries the chemical potential
    that starts the next step's mu solve: rewinding to it, or resuming it in a
    second integrator, continues bit-identically; a checkpoint of a kT = 0
    integrator is refused by a kT > 0 one and the other way round."""
    import paper_1203_6836_amd as p
    say("case fermi xlbomd checkpoint / resume 3x3x2 kT=0.5")
    m = synth.MD_MODEL
    pos = synth.lattice_positions((3, 3, 2), seed=4)
    nat = len(pos)
    vel = synth.maxwell_velocities(nat, 300.0, m.mass, seed=11)
    # zero start charges without an SCF: q - n stays large, so the divergence
    # check is off (the replay, not the physics, is under test)
    kw = dict(sp2_opts=p.options("fp64"), kT=0.5, fermi_steps=16, kappa=p.KAPPA_FINITE_T, diverge_q=0.0)
    md = ctx.xlbomd_create(m, pos, vel, np.zeros(nat), scf_max_iter=0, **kw)
    md.xlbomd_run(4)
    ck = md.xlbomd_get_state()
    assert len(ck) >= p.XL_CHECKPOINT_HEADER
    mu = np.frombuffer(ck[40:48], dtype=np.float64)[0]
    assert np.isfinite(mu)
    a = md.xlbomd_run(6)
    xa = md.xlbomd_get()
    md.xlbomd_set_state(ck)
    b = md.xlbomd_run(6)
    xb = md.xlbomd_get()
    md2 = ctx.xlbomd_create(m, pos + 0.03, np.zeros_like(vel), np.zeros(nat), scf_max_iter=0, **kw)
    md2.xlbomd_set_state(ck)
    c = md2.xlbomd_run(6)
    xc = md2.xlbomd_get()
    assert a == b == c
    for u, v, w in zip(xa, xb, xc):
        assert np.array_equal(u, v) and np.array_equal(u, w)
    md0 = ctx.xlbomd_create(m, pos, vel, np.zeros(nat), sp2_opts=p.options("fp64"), scf_max_iter=0,
                            diverge_q=0.0)
    ck0 = md0.xlbomd_get_state()
    for target, state in ((md, ck0), (md0, ck)):
        with pytest.raises(p.Sp2Error) as ei:
            target.xlbomd_set_state(state)
        assert ei.value.status == p.SP2_EINVAL
    md3 = ctx.xlbomd_create(m, pos, vel, np.zeros(nat), scf_max_iter=0, **{**kw, "fermi_steps": 14})
    with pytest.raises(p.Sp2Error) as ei:
        md3.xlbomd_set_state(ck)
    assert ei.value.status == p.SP2_EINVAL
    for h in (md, md2, md0, md3):
        h.close()


def test_finite_temperature_xlbomd_2048_orbitals_newton_passes(ctx):
    """XL-BOMD at kT = 0.5 eV on a 512-atom lattice (N = 2048) with the
    default trace tolerance, which scales with N above the floor X_0 sets:
    every step completes, and after the first the mu solve started from the
    previous step's mu takes few passes."""
    import paper_1203_6836_amd as p
    say("case fermi xlbomd 8x8x8 kT=0.5, 6 steps")
    m = synth.MD_MODEL
    dims = (8, 8, 8)
    pos = synth.lattice_positions(dims, seed=23)
    nat = len(pos)
    vel = synth.maxwell_velocities(nat, 300.0, m.mass, seed=24)
    # the charge-ordered state's gap (about 18 eV) is far above kT: the SCF
    # from the +-4 e checkerboard converges as at zero temperature
    md = ctx.xlbomd_create(m, pos, vel, synth.checkerboard_charges(dims), sp2_opts=p.options("fp64"), kT=0.5,
                           fermi_steps=16, kappa=p.KAPPA_FINITE_T, scf_beta=1.0, scf_tol=1e-7, scf_max_iter=100)
    it, res = md.xlbomd_info()
    rec = md.xlbomd_run(6)
    md.close()
    passes = [r["sp2_iterations"] for r in rec]
    say(f"  SCF {it} iterations (res {res:.1e}); Newton passes per step {passes}, "
        f"max|q-n| {max(r['max_q_minus_n'] for r in rec):.1e}")
    assert max(passes[1:]) <= 8


@pytest.mark.parametrize("n", [1, 31, 33, 101, 130, 545, 1055, 2050])
def test_product_tiles_at_ragged_sizes(ctx, n):
    """The FP64 products of the transforms at sizes around their tiles (odd
    leading dimensions, one row past a tile, both K splits): the full and
    symmetric products of a non-orthogonal FP64 solve and the recursion's, on
    random symmetric matrices, against numpy.  Bars: FP64 rounding of N-term
    sums through a 7-step factor and an 8-step recursion, far below 1e-10."""
    import paper_1203_6836_amd as p
    say(f"case ragged FP64 products N={n}")
    rng = np.random.default_rng(n)
    A = rng.standard_normal((n, n))
    H = 0.5 * (A + A.T) / np.sqrt(max(n, 2))
    e, v = np.linalg.eigh(H)
    mu, kT, steps = 0.1, 0.3, 8
    y = (e - mu) / kT / 2.0 ** (steps + 2)
    f = 1.0 / (1.0 + ((0.5 + y) / (0.5 - y)) ** (2.0 ** steps))
    D, _, _ = ctx.sp2_fermi_density_matrix(to_dev(H), 1.0, kT, steps, mu=mu, max_newton=0)
    D = D.cpu().numpy()
    err = float(np.abs(D - (v * f) @ v.T).max())
    say(f"  recursion max|dD| {err:.1e}")
    assert np.array_equal(D, D.T) and err < 1e-10
    if n < 2 or n > 1100:
        return
    B = rng.standard_normal((n, n))
    S = np.eye(n) + 0.1 * (B + B.T) / np.sqrt(n)
    n_occ = n // 2
    w, u = np.linalg.eigh(S)
    Z = (u / np.sqrt(w)) @ u.T
    Hp = Z @ H @ Z
    _, vp = np.linalg.eigh(0.5 * (Hp + Hp.T))
    ref = Z @ (vp[:, :n_occ] @ vp[:, :n_occ].T) @ Z
    R, _, _ = ctx.sp2_density_matrix_nonorth(to_dev(H), to_dev(S), n_occ, p.options("fp64"))
    err = float(np.abs(R.cpu().numpy() - ref).max())
    say(f"  non-orthogonal max|dD| {err:.1e}")
    assert err < 1e-10


@pytest.mark.parametrize("n,kT", [(1, 0.5), (2, 0.3), (33, 40.0), (101, 2.0), (130, 0.6), (530, 0.2), (530, 4.0), (1056, 0.1)])
def test_entropy_moments_at_ragged_sizes(ctx, n, kT):
    """The entropy's moments for every number of stored polynomials the
    coefficient count selects (from 2 to the most, 32) and sizes around the
    dot kernel's tiles, on random symmetric matrices against the eigenvalues:
    the moments are FP64 sums, so the bar of the lattice test applies.  The
    coefficients fall by a + sqrt(1 + a^2), a = pi kT / w over the Gershgorin half
    width w; where more than 4000 of them stay above 1e-13 the call is refused."""
    import paper_1203_6836_amd as p
    say(f"case entropy moments N={n} kT={kT}")
    rng = np.random.default_rng(100 + n)
    A = rng.standard_normal((n, n))
    H = 0.5 * (A + A.T)
    e = np.linalg.eigvalsh(H)
    mu = 0.2
    S_ref = fermi.entropy(fermi.fermi_occupations(e, mu, 1.0 / kT))
    lo, hi = osp2.gershgorin(H)
    if hi > lo and -np.log(1e-13) / np.arcsinh(2.0 * np.pi * kT / (hi - lo)) > 4200:
        with pytest.raises(p.Sp2Error) as ei:
            ctx.sp2_fermi_entropy(to_dev(H), mu, kT)
        assert ei.value.status == p.SP2_EINVAL
        return
    S, m = ctx.sp2_fermi_entropy(to_dev(H), mu, kT)
    say(f"  S {S:.12f} (eigenvalues {S_ref:.12f}), {m} coefficients")
    assert abs(S - S_ref) < 1e-10 * max(S_ref, 1.0)


@pytest.mark.parametrize("n,kT,steps,max_newton", [(1, 0.5, 12, 0), (33, 30.0, 6, 50), (101, 6.0, 8, 0),
                                                   (101, 6.0, 8, 50), (130, 3.0, 3, 50), (530, 12.0, 16, 50),
                                                   (1056, 9.0, 16, 50), (530, 1.0, 16, 50)])
def test_expansion_is_the_recursions_function(ctx, n, kT, steps, max_newton):
    """D on random symmetric matrices against the recursion's own function of
    the eigenvalues, X_n(e) = (1 - t)^(2^n) / ((1 - t)^(2^n) + (1 + t)^(2^n)) at the
    mu returned (few steps: far from the Fermi function), at a fixed and at
    the canonical mu, for coefficient counts from a handful to those where the
    recursion is used instead.  Bars: the recursion's rounding floor, 1e-10, and
    the requested trace.  A canonical solve whose bracket, the Gershgorin
    interval and 40 kT on each side, is wider than 2^(n + 1) kT is refused."""
    import paper_1203_6836_amd as p
    say(f"case fermi expansion N={n} kT={kT} steps={steps} newton={max_newton}")
    rng = np.random.default_rng(200 + n)
    A = rng.standard_normal((n, n))
    H = 0.5 * (A + A.T)
    e, v = np.linalg.eigh(H)
    n_occ, tol = max(0.37 * n, 0.3), 1e-8
    lo, hi = osp2.gershgorin(H)
    if max_newton and hi - lo + 80.0 * kT > 2.0 ** (steps + 1) * kT:
        with pytest.raises(p.Sp2Error) as ei:
            ctx.sp2_fermi_density_matrix(to_dev(H), n_occ, kT, steps, max_newton=max_newton, tol=tol)
        assert ei.value.status == p.SP2_EINVAL
        return
    D, mu, passes = ctx.sp2_fermi_density_matrix(to_dev(H), n_occ, kT, steps, mu=0.1 if max_newton == 0 else None,
                                                 max_newton=max_newton, tol=tol)
    D = D.cpu().numpy()
    t = (e - mu) / kT / 2.0 ** (steps + 1)
    f = 1.0 / (1.0 + np.exp(2.0 ** (steps + 1) * np.arctanh(t)))
    err = float(np.abs(D - (v * f) @ v.T).max())
    say(f"  mu {mu:.10f}, passes {passes}, recursion products {ctx.last_fermi_products}, max|dD| {err:.1e}")
    assert np.array_equal(D, D.T) and err < 1e-10
    assert passes * 2 * steps <= ctx.last_fermi_products <= passes * 10 * steps
    if max_newton:
        assert abs(np.trace(D) - n_occ) < 1.01 * tol


@pytest.mark.parametrize("N,kT,mu", [(45, 1e7, None), (45, 0.5, -19.0), (500, 1e7, None), (500, 0.5, None)])
def test_density_is_exactly_symmetric(ctx, N, kT, mu):
    """H symmetric only to 5e-13 of its largest element (the check's bound is
    1e-12) still gives an exactly symmetric D: where two polynomials carry the
    Fermi function (kT = 1e7), at a fixed mu far below the spectrum, and where
    products of the stored polynomials carry it."""
    rng = np.random.default_rng(N)
    H = rng.uniform(-1.0, 1.0, (N, N)) / np.sqrt(N)
    H = (H + H.T) / 2 + np.diag(np.where(np.arange(N) % 2 == 0, -2.0, 2.0))
    lower = np.tril(rng.uniform(-5e-13, 5e-13, (N, N)) * np.abs(H).max(), -1)
    say(f"case symmetric D N={N} kT={kT}")
    kw = {"max_newton": 0, "mu": mu} if mu is not None else {"tol": 1e-8}
    D, m, _ = ctx.sp2_fermi_density_matrix(to_dev(H + lower), N / 2.0, kT, 16, **kw)
    D = D.cpu().numpy()
    Dd = fermi.fermi_density(H, N / 2.0, kT, solver="lapack")[0] if mu is None else None
    assert np.array_equal(D, D.T)
    if Dd is not None:
        assert np.abs(D - Dd).max() < 1e-8


def test_expansion_gives_its_matrices_back(ctx):
    """N = 3400: the stored polynomials of the expansion take 3.1 GB during a
    call; after it the context keeps at most 2 GiB (the recursion's five
    matrices would be 0.46 GB), and a second call gives the same D."""
    import torch
    import paper_1203_6836_amd as p
    N = 3400
    say(f"case fermi work matrices N={N}")
    rng = np.random.default_rng(N)
    H = rng.uniform(-1.0, 1.0, (N, N)) / np.sqrt(N)
    Hd = to_dev((H + H.T) / 2 + np.diag(np.where(np.arange(N) % 2 == 0, -2.0, 2.0)))
    out = [torch.empty_like(Hd) for _ in range(2)]
    c = p.Context(0)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    kept = []
    for D in out:
        c.sp2_fermi_density_matrix(Hd, N / 2.0, 0.3, 16, tol=1e-7, D_out=D)
        c.sp2_fermi_entropy(Hd, 0.0, 0.3)
        kept.append(free0 - torch.cuda.mem_get_info()[0])
    say(f"  kept {kept}")
    c.close()
    assert max(kept) <= (2 << 30) + (64 << 20)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("kT,steps,kw,recursion", [(0.5, 16, {"tol": 1e-8}, False),
                                                   (0.25, 16, {"max_newton": 0, "mu": -5.0}, True),
                                                   (0.5, 8, {"tol": 4e-11}, True)])
def test_products_formed_tell_the_path(ctx, kT, steps, kw, recursion):
    """N = 108: the recursion launches exactly the products of its count (a
    fixed mu at kT = 0.25 eV, where one pass is cheaper than the expansion, and
    a tol below 4e-13 N), the expansion less than half of them; both give the
    function that the recursion defines, 1 / (1 + exp(2^(n + 1) atanh t)) with
    t = (e - mu) / (kT 2^(n + 1))."""
    w, H = lattice((3, 3, 3), 7)
    Hd = to_dev(H)
    say(f"case products formed kT={kT} {kw}")
    D, mu, passes = ctx.sp2_fermi_density_matrix(Hd, w.n_occ, kT, steps, **kw)
    formed, counted = ctx.sp2_fermi_products_formed(), ctx.last_fermi_products
    say(f"  formed {formed}, the recursion's {counted} in {passes} passes")
    e, v = np.linalg.eigh(H)
    t = (e - mu) / kT / 2.0 ** (steps + 1)
    f = 1.0 / (1.0 + np.exp(2.0 ** (steps + 1) * np.arctanh(t)))
    assert np.abs(D.cpu().numpy() - (v * f) @ v.T).max() < 1e-9
    if recursion:
        assert formed == counted
    else:
        assert 0 < formed < counted / 2
    ctx.sp2_fermi_entropy(Hd, mu, kT)
    assert 0 < ctx.sp2_fermi_products_formed() < counted / 2 or recursion
