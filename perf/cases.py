"""The work that users of the library bring to it, as measurable cases.

A case is a call sequence on one system of the synthetic tight-binding model
(jittered simple-cubic clusters with four orbitals per atom, N = 4 atoms; the
gapped wire for the thresholded solver), through the binding's entry points:

  evaluate  one Born-Oppenheimer evaluation: H[n], D, charges, energies, forces
  solve     density matrix by SP2 of a dense H on the device, then its charges
            and band energy (FP64, or int8 digit planes with the benchmark's
            or the library's default recipe)
  wire      the same with the elementwise threshold (linear-scaling regime)
  nonorth   density matrix in a non-orthogonal basis, and its charges
  fermi     finite electronic temperature: D at the canonical mu, and the entropy
  xlbomd    extended-Lagrangian MD steps resumed from a checkpoint
  serve     a burst of solves of uneven sizes through the batching server,
            host arrays in and out

``exact`` is plain torch in float64: eigenpairs on the host up to N = 2048,
above that the definition's purification with torch's own matrix products.
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

import paper_1203_6836_amd as lib

# ------------------------------------------------------------ the model
_BASE = dict(eps_s=-8.0, eps_p=-4.0, t0=2.0, r0=1.5, lam=0.5, r_cut=4.0, r_tail=4.0, hubbard_u=4.0,
             coulomb_k=14.399645478, pair_a=0.0, pair_r0=1.5, pair_rho=0.3, mass=12.0, z_val=4,
             overlap_s0=0.0, overlap_lam=0.5)
STATIC = types.SimpleNamespace(**_BASE)
MD = types.SimpleNamespace(**{**_BASE, "r_tail": 3.5, "pair_a": 5.605396, "pair_rho": 0.15})
GAPPED = types.SimpleNamespace(**{**_BASE, "eps_p": 4.0, "z_val": 2})
NONORTH = types.SimpleNamespace(**{**_BASE, "overlap_s0": 0.05})
ACC_A_FS2 = 9.648533212e-3      # 1 eV/(A amu) in A/fs^2
KE_EV = 103.6426965             # 1 amu A^2/fs^2 in eV
KB_EV = 8.617333262e-5          # eV/K
DT_FS, KAPPA, ALPHA = 0.25, 0.91, 0.018
DISSIPATION = (-6.0, 14.0, -8.0, -3.0, 4.0, -1.0)
TAU = 1e-5


def _sites(dims, count):
    nx, ny, nz = dims
    iz, iy, ix = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    return np.stack([ix.ravel(), iy.ravel(), iz.ravel()], axis=1)[:count].astype(np.float64)


def _positions(case, seed):
    """Jittered lattice of the case, x fastest: a box, or the first atoms of a cube."""
    if case["path"] == "wire":
        dims, spacing = (4, 4, case["layers"]), 2.0
    elif case["path"] == "xlbomd":
        dims, spacing = tuple(int(d) for d in case["box"].split("x")), 1.5
    else:
        side = int(math.ceil(round(case["atoms"] ** (1.0 / 3.0), 9)))
        dims, spacing = (side, side, side), 1.5
    count = case.get("atoms") or dims[0] * dims[1] * dims[2]
    sites = _sites(dims, count)
    rng = np.random.default_rng([seed, 7])
    return sites * spacing + rng.normal(0.0, 0.1, sites.shape), sites


def _radial(r, amp, r0, decay, r1, rcut):
    """amp exp(-(r - r0)/decay) up to r1, a quintic to zero at rcut (value, slope, curvature)."""
    f = amp * torch.exp(-(r - r0) / decay)
    if r1 < rcut:
        z = amp * math.exp(-(r1 - r0) / decay)
        b0, b1, b2, d = z, -z / decay, 0.5 * z / decay ** 2, rcut - r1
        rhs = np.array([-(b0 + b1 * d + b2 * d * d), -(b1 + 2 * b2 * d), -2 * b2])
        mat = np.array([[d ** 3, d ** 4, d ** 5], [3 * d ** 2, 4 * d ** 3, 5 * d ** 4],
                        [6 * d, 12 * d ** 2, 20 * d ** 3]])
        b3, b4, b5 = np.linalg.solve(mat, rhs)
        x = r - r1
        f = torch.where(r < r1, f, b0 + x * (b1 + x * (b2 + x * (b3 + x * (b4 + x * b5)))))
    return torch.where(r < rcut, f, torch.zeros_like(f))


def _pairs(pos):
    """Pair vectors' unit components and distances (the diagonal's distance is 1e9)."""
    d = [pos[None, :, k] - pos[:, None, k] for k in range(3)]
    eye = torch.eye(len(pos), dtype=pos.dtype, device=pos.device)
    r = torch.sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + eye * 1e18)
    return [x / r for x in d], r


def _blocks(c, t):
    """The Slater-Koster matrix of magnitude t: ss -t, sp +t, pp-sigma +t, pp-pi -t."""
    n = len(t)
    out = t.new_empty((n, 4, n, 4))
    out[:, 0, :, 0] = -t
    for k in range(3):
        out[:, 0, :, k + 1] = c[k] * t
        out[:, k + 1, :, 0] = -c[k] * t
        for l in range(3):
            out[:, k + 1, :, l + 1] = 2.0 * t * (c[k] * c[l]) - (t if k == l else 0.0)
    return out.reshape(4 * n, 4 * n)


def _hamiltonian(pos, m, shift=None):
    """H = h + diag(shift) as float64 torch, on pos's device."""
    c, r = _pairs(pos)
    h = _blocks(c, _radial(r, m.t0, m.r0, m.lam, m.r_tail, m.r_cut))
    onsite = pos.new_tensor([m.eps_s, m.eps_p, m.eps_p, m.eps_p]).repeat(len(pos))
    if shift is not None:
        onsite = onsite + shift.repeat_interleave(4)
    h.diagonal().add_(onsite)
    return h


def _overlap(pos, m):
    c, r = _pairs(pos)
    s = -_blocks(c, _radial(r, m.overlap_s0, m.r0, m.overlap_lam, m.r_tail, m.r_cut))
    s.diagonal().add_(1.0)
    return s


def _potential(pos, n, m):
    _, r = _pairs(pos)
    return (m.coulomb_k / r) @ n + m.hubbard_u * n - m.coulomb_k * 1e-9 * n


def _n_occ(case, atoms):
    return atoms if case["path"] == "wire" else 2 * atoms


# ------------------------------------------------------------ the library side
_CTX = None


def _context():
    """One context per process, as a program keeps one."""
    global _CTX
    if _CTX is None:
        _CTX = lib.Context(0)
    return _CTX


def _options(case):
    kw = {}
    if case["precision"] == "int8x":
        kw.update(slices=case["slices"], levels=case["levels"])
    if case["path"] == "wire":
        kw.update(tau=TAU, threshold=1)
    return lib.options(case["precision"], **kw)


def _serve_sizes(case, seed):
    return np.random.default_rng([case["size_seed"], 11]).integers(32, case["max_atoms"] + 1, case["requests"])


def _velocities(atoms, seed):
    rng = np.random.default_rng([seed, 13])
    v = rng.normal(0.0, math.sqrt(KB_EV * 300.0 / (12.0 * KE_EV)), (atoms, 3))
    return v - v.mean(axis=0, keepdims=True)


def _aux_charges(atoms, seed):
    return np.random.default_rng([seed, 17]).uniform(-0.2, 0.2, atoms)


def _mu_tol(n):
    return 1e-9 * max(1.0, n / 512.0)     # the integrator's default bound on |Tr D - n_occ|


def prepare(case, seed):
    ctx, path = _context(), case["path"]
    st = types.SimpleNamespace(case=case, ctx=ctx)
    if path == "serve":
        st.requests = []
        for k, atoms in enumerate(_serve_sizes(case, seed)):
            pos, _ = _positions({"path": "solve", "atoms": int(atoms)}, 1000 * seed + k)
            h = _hamiltonian(torch.from_numpy(pos).cuda(), STATIC).cpu().numpy()
            st.requests.append((h, 2 * int(atoms)))
        st.server = lib.Server(ctx, slices=4, levels=5)
        return st
    pos, sites = _positions(case, seed)
    atoms = len(pos)
    st.atoms, st.n_occ = atoms, _n_occ(case, atoms)
    if path == "xlbomd":
        guess = np.where(sites.sum(axis=1) % 2 == 0, 4.0, -4.0)
        st.md = ctx.xlbomd_create(MD, pos, _velocities(atoms, seed), guess, dt_fs=DT_FS, kappa=KAPPA, alpha=ALPHA,
                                  c=DISSIPATION, sp2_opts=_options(case), scf_beta=1.0, scf_tol=1e-6,
                                  scf_max_iter=100)
        st.checkpoint = st.md.xlbomd_get_state()
        return st
    xyz = torch.from_numpy(pos).cuda()
    if path == "evaluate":
        st.xyz, st.n = xyz, torch.from_numpy(_aux_charges(atoms, seed)).cuda()
        st.opts = _options(case)
    elif path == "nonorth":
        st.H, st.S, st.opts = _hamiltonian(xyz, NONORTH), _overlap(xyz, NONORTH), _options(case)
    elif path == "fermi":
        st.H = _hamiltonian(xyz, STATIC)
    else:
        st.H = _hamiltonian(xyz, GAPPED if path == "wire" else STATIC)
        st.opts = _options(case)
    return st


def run(st):
    case, ctx, path = st.case, st.ctx, st.case["path"]
    if path == "evaluate":
        q, e_band, e_pot, F, _ = ctx.qmd_evaluate(MD, st.xyz, st.n, st.n_occ, st.opts)
        return {"q": q, "e_band": e_band, "e_pot": e_pot, "F": F}
    if path in ("solve", "wire"):
        D, _ = ctx.sp2_density_matrix(st.H, st.n_occ, st.opts)
        q = ctx.sp2_mulliken(D, st.atoms, 2.0 if path == "wire" else 4.0)
        return {"D": D, "q": q, "e_band": ctx.sp2_band_energy(D, st.H)}
    if path == "nonorth":
        D, _, _ = ctx.sp2_density_matrix_nonorth(st.H, st.S, st.n_occ, st.opts)
        return {"D": D, "q": ctx.sp2_mulliken_overlap(D, st.S, st.atoms)}
    if path == "fermi":
        D, mu, _ = ctx.sp2_fermi_density_matrix(st.H, st.n_occ, case["kT"], case["steps"],
                                                tol=_mu_tol(4 * st.atoms))
        entropy, _ = ctx.sp2_fermi_entropy(st.H, mu, case["kT"])
        return {"D": D, "mu": mu, "entropy": entropy}
    if path == "xlbomd":
        st.md.xlbomd_set_state(st.checkpoint)
        log = st.md.xlbomd_run(case["md_steps"])
        xyz, vel, q, n = st.md.xlbomd_get()
        energies = np.array([[rec["etot"], rec["epot"], rec["ekin"]] for rec in log])
        return {"xyz": xyz, "vel": vel, "q": q, "n": n, "energies": energies}
    tickets = [st.server.sp2_server_submit(h, n_occ) for h, n_occ in st.requests]
    out = [st.server.sp2_server_wait(t, len(h)) for t, (h, _) in zip(tickets, st.requests)]
    return [{"D": D, "q": q} for D, q, _ in out]


# ------------------------------------------------------------ what it cannot do without
def work(case):
    """Bytes: the matrices in and out once.  Flops: the distinct entries of
    each symmetric product, N^2 (N + 1), times the products of the recursion
    (62 on the clusters, 18 on the wire, 18 per MD step, 16 squarings and as
    many inverses of the Fermi operator's one pass at the final mu)."""
    path = case["path"]
    if path == "serve":
        sizes = [4.0 * a for a in _serve_sizes(case, 0)]
        return {"bytes": sum(16.0 * n * n + 2.0 * n for n in sizes), "flops": sum(62.0 * n * n * (n + 1) for n in sizes)}
    if path == "wire":
        n = 64.0 * case["layers"]
        band = min(n, 800.0)          # columns of X_n that survive the threshold
        return {"bytes": 16.0 * n * n, "flops": 18.0 * n * band * band}
    if path == "xlbomd":
        n = 4.0 * math.prod(int(d) for d in case["box"].split("x"))
        return {"bytes": case["md_steps"] * 30.0 * n, "flops": case["md_steps"] * 18.0 * n * n * (n + 1)}
    n = 4.0 * case["atoms"]
    if path == "evaluate":
        return {"bytes": 16.0 * n, "flops": 62.0 * n * n * (n + 1)}
    if path == "nonorth":
        return {"bytes": 24.0 * n * n, "flops": (62.0 + 20.0 + 6.0) * n * n * (n + 1)}
    if path == "fermi":
        return {"bytes": 16.0 * n * n, "flops": 2.0 * case["steps"] * n * n * (n + 1)}
    return {"bytes": 16.0 * n * n, "flops": 62.0 * n * n * (n + 1)}


# ------------------------------------------------------------ exact values
def _purify(H, n_occ, tau=0.0):
    """SP2 in float64 (elementwise threshold tau), torch's own products."""
    H = H.cuda() if torch.cuda.is_available() else H
    off = H.abs().sum(1) - H.diagonal().abs()
    lo, hi = float((H.diagonal() - off).min()), float((H.diagonal() + off).max())
    X = H / -(hi - lo)
    X.diagonal().add_(hi / (hi - lo))
    cut = (lambda A: A.masked_fill_(A.abs() < tau, 0.0)) if tau > 0.0 else (lambda A: A)
    X = cut(X)
    errs = []
    for _ in range(128):
        P = X @ X
        P = 0.5 * (P + P.T)
        t1, t2 = float(X.diagonal().sum()), float(P.diagonal().sum())
        errs.append(float(torch.linalg.norm(P - X)))
        if tau > 0.0:
            floor = len(errs) > 4 and errs[-1] >= 0.5 * errs[-3] and errs[-1] < 0.1
        else:
            floor = len(errs) > 4 and errs[-1] >= errs[-3] and errs[-1] < 1e-2
        if errs[-1] < 1e-10 or floor:
            return X
        X = cut(P if abs(t2 - n_occ) <= abs(2.0 * t1 - t2 - n_occ) else P.neg_().add_(X, alpha=2.0))
    raise RuntimeError("no convergence")


def _projector(H, n_occ):
    if len(H) > 2048:
        return _purify(H, n_occ)
    _, v = torch.linalg.eigh(H.cpu())
    return v[:, :n_occ] @ v[:, :n_occ].T


def _populations(D):
    return 2.0 * D.diagonal().reshape(-1, 4).sum(1)


def _evaluation(pos, n, n_occ, m):
    """D, q, band energy, U and F = -dU/dR at constant n, D and q."""
    V = _potential(pos, n, m)
    H = _hamiltonian(pos, m, V)
    D = _projector(H, n_occ).to(H.device)
    q = _populations(D) - m.z_val
    R = pos.clone().requires_grad_(True)
    c, r = _pairs(R)
    rep = _radial(r, m.pair_a, m.pair_r0, m.pair_rho, m.r_tail, m.r_cut)
    VR = _potential(R, n, m)
    U = 2.0 * (D * _hamiltonian(R, m)).sum() + (q * VR).sum() - 0.5 * (n * VR).sum() + 0.5 * rep.sum()
    F, = torch.autograd.grad(-U, R)
    return D, q, 2.0 * float((D * H).sum()), float(U.detach()), F


def _exact_md(case, seed):
    pos, sites = _positions(case, seed)
    atoms = len(pos)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    x = torch.from_numpy(pos).to(dev)
    v = torch.from_numpy(_velocities(atoms, seed)).to(dev)
    n = torch.from_numpy(np.where(sites.sum(axis=1) % 2 == 0, 4.0, -4.0)).to(dev)
    for _ in range(100):
        D = _projector(_hamiltonian(x, MD, _potential(x, n, MD)), 2 * atoms).to(dev)
        q = _populations(D) - MD.z_val
        if float((q - n).abs().max()) < 1e-6:
            break
        n = q
    hist = [q] * len(DISSIPATION)
    _, q, _, U, F = _evaluation(x, hist[0], 2 * atoms, MD)
    half = 0.5 * DT_FS * ACC_A_FS2 / MD.mass
    energies = []
    for _ in range(case["md_steps"]):
        v = v + half * F
        x = x + DT_FS * v
        new = 2.0 * hist[0] - hist[1] + KAPPA * (q - hist[0]) + ALPHA * sum(c * h for c, h in zip(DISSIPATION, hist))
        hist = [new] + hist[:-1]
        _, q, _, U, F = _evaluation(x, new, 2 * atoms, MD)
        v = v + half * F
        kin = 0.5 * MD.mass * KE_EV * float((v * v).sum())
        energies.append([U + kin, U, kin])
    host = [t.cpu().numpy() for t in (x, v, q, hist[0])]
    return {"xyz": host[0], "vel": host[1], "q": host[2], "n": host[3], "energies": np.array(energies)}


def _exact_fermi(case, H, n_occ):
    """The n-step recursion's occupations at the canonical mu, by eigenpairs."""
    e, v = torch.linalg.eigh(H.cpu())
    kT, steps = case["kT"], case["steps"]

    def occupations(mu):
        y = (e - mu) / kT / 2.0 ** (steps + 2)
        return torch.special.expit(-(2.0 ** steps) * (torch.log1p(2.0 * y) - torch.log1p(-2.0 * y)))

    lo, hi = float(e[0]) - 40 * kT, float(e[-1]) + 40 * kT
    for _ in range(200):
        mu = 0.5 * (lo + hi)
        lo, hi = (mu, hi) if float(occupations(mu).sum()) < n_occ else (lo, mu)
    x = ((e - mu) / kT).abs()
    s = torch.log1p(torch.exp(-x)) + x * torch.exp(-x) / (1.0 + torch.exp(-x))
    return {"D": (v * occupations(mu)) @ v.T, "mu": mu, "entropy": 2.0 * float(s.sum())}


def exact(case, seed):
    path = case["path"]
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if path == "serve":
        out = []
        for k, atoms in enumerate(_serve_sizes(case, seed)):
            pos, _ = _positions({"path": "solve", "atoms": int(atoms)}, 1000 * seed + k)
            D = _projector(_hamiltonian(torch.from_numpy(pos), STATIC), 2 * int(atoms))
            out.append({"D": D.numpy(), "q": (_populations(D) - 4.0).numpy()})
        return out
    if path == "xlbomd":
        return _exact_md(case, seed)
    pos, _ = _positions(case, seed)
    atoms = len(pos)
    xyz, n_occ = torch.from_numpy(pos).to(dev), _n_occ(case, atoms)
    if path == "evaluate":
        n = torch.from_numpy(_aux_charges(atoms, seed)).to(dev)
        _, q, e_band, e_pot, F = _evaluation(xyz, n, n_occ, MD)
        return {"q": q, "e_band": e_band, "e_pot": e_pot, "F": F}
    if path == "nonorth":
        H, S = _hamiltonian(xyz, NONORTH).cpu(), _overlap(xyz, NONORTH).cpu()
        w, u = torch.linalg.eigh(S)
        Z = (u / w.sqrt()) @ u.T
        Hp = Z @ H @ Z
        D = Z @ _projector(0.5 * (Hp + Hp.T), n_occ) @ Z
        return {"D": D, "q": 2.0 * (D * S).sum(1).reshape(-1, 4).sum(1) - NONORTH.z_val}
    if path == "fermi":
        return _exact_fermi(case, _hamiltonian(xyz, STATIC), n_occ)
    if path == "wire":
        H = _hamiltonian(xyz, GAPPED)
        D, z = _purify(H, n_occ, TAU), 2.0
    else:
        H = _hamiltonian(xyz, STATIC)
        D, z = _projector(H, n_occ), 4.0
    H = H.to(D.device)
    return {"D": D, "q": _populations(D) - z, "e_band": 2.0 * float((D * H).sum())}


# ------------------------------------------------------------ the cases
def listed():
    bench = dict(precision="int8x", slices=4, levels=5)     # the benchmark's digit recipe
    default = dict(precision="int8x", slices=5, levels=0)   # the library's
    fp64 = dict(precision="fp64")
    return [
        # the smallest system the request stream holds, everything an MD driver asks of one geometry
        dict(name="evaluate_fp64_n128", path="evaluate", atoms=32, **fp64),
        # a ragged mid-size FP64 solve (N is no multiple of a tile)
        dict(name="solve_fp64_n1020", path="solve", atoms=255, **fp64),
        # FP64 at the size of the 1024-atom MD system
        dict(name="solve_fp64_n4096", path="solve", atoms=1024, **fp64),
        # a ragged small solve with the benchmark's recipe
        dict(name="solve_int8_n720", path="solve", atoms=180, **bench),
        # the library's default int8 recipe at the largest request size
        dict(name="solve_int8_n2048", path="solve", atoms=512, **default),
        # the benchmark's solve: the largest dense system in use
        dict(name="solve_int8_n8192", path="solve", atoms=2048, **bench),
        # the paper's threshold on an insulator: 4096 atoms in the linear-scaling regime
        dict(name="wire_int8_n16384", path="wire", layers=256, **bench),
        # a non-orthogonal density matrix, ragged
        dict(name="nonorth_int8_n2000", path="nonorth", atoms=500, **bench),
        # electronic temperature, small and ragged (a cluster) and large
        dict(name="fermi_n500", path="fermi", atoms=125, kT=0.5, steps=16),
        dict(name="fermi_n2048", path="fermi", atoms=512, kT=0.5, steps=16),
        # MD of the 1024-atom box, resumed from a checkpoint
        dict(name="xlbomd_int8_n4096", path="xlbomd", box="8x8x16", md_steps=2, **bench),
        # a burst on the server: sizes uniform in 32-512 atoms as in the request stream
        dict(name="serve_int8_24", path="serve", requests=24, max_atoms=512, size_seed=5),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["evaluate", "solve", "solve", "solve", "wire", "nonorth", "fermi", "xlbomd", "serve"])
    recipes = [dict(precision="fp64"), dict(precision="int8x", slices=4, levels=5),
               dict(precision="int8x", slices=5, levels=0)]
    if path == "evaluate":
        return dict(path=path, atoms=_spread(rng, 27, 512), **rng.choice(recipes))
    if path == "solve":
        recipe = rng.choice(recipes)
        return dict(path=path, atoms=_spread(rng, 32, 1024 if recipe["precision"] == "fp64" else 2048), **recipe)
    if path == "wire":
        return dict(path=path, layers=_spread(rng, 16, 256), **rng.choice(recipes[1:]))
    if path == "nonorth":
        return dict(path=path, atoms=_spread(rng, 27, 512), **rng.choice(recipes))
    if path == "fermi":
        return dict(path=path, atoms=_spread(rng, 27, 512), kT=rng.choice([0.25, 0.5, 1.0]), steps=16)
    if path == "xlbomd":
        box = rng.choice(["4x4x4", "4x4x6", "4x6x6", "6x6x6", "6x6x8", "6x8x8", "8x8x8", "8x8x10", "8x8x16"])
        return dict(path=path, box=box, md_steps=rng.choice([1, 2, 4]), **rng.choice(recipes))
    return dict(path=path, requests=rng.randint(4, 24), max_atoms=_spread(rng, 64, 512), size_seed=rng.randint(1, 99))
