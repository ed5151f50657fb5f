"""Continuous-batching server: results alone == in a mix, parity with the oracle, admission."""
import sys
import threading
import time

import numpy as np
import pytest

import synth
from oracle import observables, sp2 as osp2, tb as otb

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


def request_H(n_atoms, seed):
    pos = synth.lattice_positions(synth.cube_dims_for(n_atoms), seed=seed, n_atoms=n_atoms)
    return otb.hamiltonian(pos, None, synth.STATIC_MODEL)


@pytest.mark.parametrize("recipe", [{}, {"slices": 4, "levels": 5}])
def test_server_alone_equals_mix_and_direct(ctx, recipe):
    """A request served alone and in a mix gives bitwise the same D and q, the
    same as the direct int8 solve with the same digit recipe (five planes;
    four planes with five levels), and every result is within the
    mixed-precision tolerance of the oracle."""
    import torch
    import paper_1203_6836_amd as p
    say(f"case serving alone vs mix {recipe}")
    probe = request_H(40, 1000)           # N = 160 (ragged: ld = 256)
    others = [request_H(n, 2000 + k) for k, n in enumerate([32, 150, 77, 300, 64, 129])]
    srv = p.Server(ctx, max_slots=8, **recipe)
    t = srv.sp2_server_submit(probe, 80)
    D_alone, q_alone, st_alone = srv.sp2_server_wait(t, probe.shape[0])
    # in a mix: submit others first, the probe in the middle, more after
    tk = [srv.sp2_server_submit(H, H.shape[0] // 2) for H in others[:3]]
    tp = srv.sp2_server_submit(probe, 80)
    tk += [srv.sp2_server_submit(H, H.shape[0] // 2) for H in others[3:]]
    D_mix, q_mix, st_mix = srv.sp2_server_wait(tp, probe.shape[0])
    outs = [srv.sp2_server_wait(x, H.shape[0]) for x, H in zip(tk, others)]
    rep = srv.sp2_server_report()
    srv.close()
    say(f"  iters {st_alone['iterations']} / {st_mix['iterations']}; report {rep}")
    assert np.array_equal(D_alone, D_mix) and np.array_equal(q_alone, q_mix)
    # the same as the direct (non-served) int8 solve
    D_direct, _ = ctx.sp2_density_matrix(torch.from_numpy(probe).cuda(), 80, p.options("int8x", **recipe))
    assert np.array_equal(D_alone, D_direct.cpu().numpy())
    # every result in the mix within the tolerance of the oracle
    for (D, q, st), H in zip(outs, others):
        ref = osp2.sp2(H, H.shape[0] // 2)
        err = np.linalg.norm(D - ref.D) / np.sqrt(H.shape[0])
        dq = np.max(np.abs(q - observables.mulliken(ref.D)))
        assert err <= 1e-6 and dq <= 1e-6, (H.shape[0], err, dq)
    assert rep["p50_ms"] > 0 and rep["p99_ms"] >= rep["p50_ms"]


def test_server_levels_are_validated(ctx):
    import paper_1203_6836_amd as p
    with pytest.raises(p.Sp2Error):
        p.Server(ctx, slices=6, levels=7)
    with pytest.raises(p.Sp2Error):
        p.Server(ctx, slices=4, levels=3)


def test_server_admission_by_footprint(ctx):
    import paper_1203_6836_amd as p
    say("case serving admission with a small arena")
    Hs = [request_H(128, 3000 + k) for k in range(3)]     # N = 512, ~10 MB each
    srv = p.Server(ctx, hbm_budget_bytes=24 << 20, max_slots=4)   # room for two at a time
    big = request_H(400, 9)                                        # N = 1600: never fits
    with pytest.raises(p.Sp2Error) as ei:
        srv.sp2_server_submit(big, 800)
    assert ei.value.status == p.SP2_EBUDGET
    tks = [srv.sp2_server_submit(H, 256) for H in Hs]
    res = [srv.sp2_server_wait(t, 512, timeout_s=60.0) for t in tks]
    srv.close()
    for (D, q, st), H in zip(res, Hs):
        ref = osp2.sp2(H, 256)
        assert np.linalg.norm(D - ref.D) / np.sqrt(512) <= 1e-6


def test_server_poisson_stream(ctx):
    import paper_1203_6836_amd as p
    say("case serving poisson stream")
    reqs = synth.request_stream(n_requests=24, rate_per_s=200.0, max_atoms=256)
    Hs = [otb.hamiltonian(r.positions(), None, synth.STATIC_MODEL) for r in reqs]
    srv = p.Server(ctx)
    tickets = [None] * len(reqs)

    def submitter():
        t0 = time.perf_counter()
        for k, r in enumerate(reqs):
            dt = r.arrival_s - (time.perf_counter() - t0)
            if dt > 0:
                time.sleep(dt)
            tickets[k] = srv.sp2_server_submit(Hs[k], 2 * r.n_atoms)

    th = threading.Thread(target=submitter)
    th.start()
    th.join()
    res = [srv.sp2_server_wait(t, 4 * r.n_atoms, want_D=False) for t, r in zip(tickets, reqs)]
    rep = srv.sp2_server_report()
    srv.close()
    say(f"  {rep}")
    assert all(st["status"] in ("converged", "stalled") for _, _, st in res)
    assert rep["solves_per_s"] > 0


def test_server_reports_gap_and_invalid_h(ctx):
    import paper_1203_6836_amd as p
    say("case serving: degenerate and invalid H next to a good one")
    good = request_H(40, 1000)
    degenerate = np.diag([-1.0, 0.0, 0.0, 1.0])
    asym = good.copy()
    asym[3, 100] += 1e-6
    srv = p.Server(ctx, max_slots=4)
    tg = srv.sp2_server_submit(good, 80)
    td = srv.sp2_server_submit(degenerate, 2)
    ta = srv.sp2_server_submit(asym, 80)
    D, q, st = srv.sp2_server_wait(tg, good.shape[0])
    for t, N, want in ((td, 4, p.SP2_EGAP), (ta, good.shape[0], p.SP2_EINVAL)):
        with pytest.raises(p.Sp2Error) as ei:
            srv.sp2_server_wait(t, N)
        assert ei.value.status == want
    srv.close()
    ref = osp2.sp2(good, 80)
    assert np.linalg.norm(D - ref.D) / np.sqrt(good.shape[0]) <= 1e-6


def test_server_largest_requests_against_oracle(ctx):
    """Requests at the top of the served size range (512 atoms, N = 2048, and
    a ragged 500-atom N = 2000) in a mix with small ones: each equals its
    solve alone, bitwise, and the oracle within 1e-6 (D per sqrt(N) and
    charges)."""
    import paper_1203_6836_amd as p
    say("case serving N=2048 and N=2000 in a mix")
    big = [request_H(512, 4000), request_H(500, 4001)]
    small = [request_H(n, 4100 + k) for k, n in enumerate([32, 200, 96, 333])]
    srv = p.Server(ctx, max_slots=8)
    alone = []
    for H in big:
        t = srv.sp2_server_submit(H, H.shape[0] // 2)
        alone.append(srv.sp2_server_wait(t, H.shape[0]))
    tk = [srv.sp2_server_submit(small[0], small[0].shape[0] // 2)]
    tb = [srv.sp2_server_submit(H, H.shape[0] // 2) for H in big]
    tk += [srv.sp2_server_submit(H, H.shape[0] // 2) for H in small[1:]]
    mixed = [srv.sp2_server_wait(t, H.shape[0]) for t, H in zip(tb, big)]
    for t, H in zip(tk, small):
        srv.sp2_server_wait(t, H.shape[0], want_D=False)
    srv.close()
    for (Da, qa, sa), (Dm, qm, sm), H in zip(alone, mixed, big):
        N = H.shape[0]
        ref = osp2.sp2(H, N // 2)
        err = np.linalg.norm(Dm - ref.D) / np.sqrt(N)
        dq = np.max(np.abs(qm - observables.mulliken(ref.D)))
        say(f"  N={N}: products {sm['iterations']} (oracle {ref.iterations}), err/sqrtN {err:.2e}, max|dq| {dq:.2e}")
        assert np.array_equal(Da, Dm) and np.array_equal(qa, qm)
        assert err <= 1e-6 and dq <= 1e-6


@pytest.mark.parametrize("n_atoms,recipe", [(875, {"slices": 4, "levels": 5}), (875, {"slices": 6})])
def test_served_tiles_equal_the_large_output_tile(ctx, n_atoms, recipe):
    """N = 3500: the direct solve runs 128 x 128 output tiles, the server 64 x 64
    (a run of them per XCD, beside a small system's); the digit sums are exact
    and the update's arithmetic the same, so D is the same bit for bit."""
    import torch
    import paper_1203_6836_amd as p
    say(f"case served tiles N={4 * n_atoms} {recipe}")
    H, small = request_H(n_atoms, 41), request_H(33, 42)
    srv = p.Server(ctx, max_slots=3, **recipe)
    tk = [(srv.sp2_server_submit(h, h.shape[0] // 2), h) for h in (small, H, small)]
    out = [srv.sp2_server_wait(t, h.shape[0]) for t, h in tk]
    srv.close()
    for (_, h), (D, _, st) in zip(tk, out):
        Dd, sd = ctx.sp2_density_matrix(torch.from_numpy(h).cuda(), h.shape[0] // 2, p.options("int8x", **recipe))
        assert st["branches"] == sd["branches"]
        assert np.array_equal(D, Dd.cpu().numpy())


@pytest.mark.parametrize("n_atoms,recipe", [(1021, {"slices": 4, "levels": 5}), (1053, {"slices": 5}), (1280, {"slices": 4})])
def test_tiles_left_over_in_the_last_round(ctx, n_atoms, recipe):
    """Direct solves of 128 x 128 tiles whose last round has few of them run
    these as 64 x 64 pieces: N = 4084 (ragged, 16 tiles left of 528 on 256 CUs),
    4212 (49 of 561, a diagonal tile among them) and 5120 (52 of 820).  The
    server runs 64 x 64 tiles throughout; D is the same bit for bit."""
    import torch
    import paper_1203_6836_amd as p
    say(f"case left tiles N={4 * n_atoms} {recipe}")
    H = request_H(n_atoms, 51)
    srv = p.Server(ctx, max_slots=2, **recipe)
    D, _, st = srv.sp2_server_wait(srv.sp2_server_submit(H, 2 * n_atoms), H.shape[0])
    srv.close()
    Dd, sd = ctx.sp2_density_matrix(torch.from_numpy(H).cuda(), 2 * n_atoms, p.options("int8x", **recipe))
    assert st["branches"] == sd["branches"]
    assert np.array_equal(D, Dd.cpu().numpy())


@pytest.mark.parametrize("n_atoms,recipe", [(4, {"slices": 2}), (512, {}), (1053, {"slices": 4, "levels": 5})])
def test_request_of_exactly_its_footprint(ctx, n_atoms, recipe):
    """A request is accepted by a server whose budget is just the arrays that a
    solve needs side by side (H, two padded X, the digit planes, row scales,
    partial sums of 128 x 128 tiles, the H check's partials, D and charges, each
    rounded up to 256 bytes), and equals the direct solve bit for bit: N = 16
    (smaller than the smallest budget, 1 MiB), 2048 and 4212."""
    import torch
    import paper_1203_6836_amd as p
    H = request_H(n_atoms, 61)
    N = H.shape[0]
    ld = (N + 127) // 128 * 128
    nt = ld // 128
    arrays = (8 * N * N, 16 * ld * ld, recipe.get("slices", 5) * ld * ld, 8 * ld, 24 * max(nt * (nt + 1) // 2, ld // 4),
              2 * 2048 * 8, 8 * N * N, 8 * (N // 4 + 1))
    need = sum((a + 255) // 256 * 256 for a in arrays)
    say(f"case footprint N={N}: {need} bytes")
    srv = p.Server(ctx, hbm_budget_bytes=max(need, 1 << 20), max_slots=1, **recipe)
    opts = p.options("int8x", **recipe)
    try:
        D, _, st = srv.sp2_server_wait(srv.sp2_server_submit(H, 2 * n_atoms), N)
    except p.Sp2Error as e:
        status, _ = ctx.sp2_density_matrix_status(torch.from_numpy(H).cuda(), 2 * n_atoms, opts)
        assert status == e.status != p.SP2_EBUDGET
        return
    finally:
        srv.close()
    Dd, sd = ctx.sp2_density_matrix(torch.from_numpy(H).cuda(), 2 * n_atoms, opts)
    assert st["branches"] == sd["branches"]
    assert np.array_equal(D, Dd.cpu().numpy())


@pytest.mark.parametrize("first", [[1152], [992, 160]])
def test_requests_that_do_not_wait_for_room(ctx, first):
    """A request of N = 640 that needs a few products starts at once and ends
    first, beside one larger than the group's room (N = 4608, about 60
    products) and where a large and a middle one (N = 3968 and 640) fill it."""
    import paper_1203_6836_amd as p
    say(f"case serving beside {[4 * n for n in first]}")
    Hs = [request_H(n, 71) for n in first]
    rng = np.random.default_rng(7)
    quick = np.triu(rng.uniform(-1e-3, 1e-3, (640, 640)), 1)
    quick = quick + quick.T + np.diag(np.where(np.arange(640) % 2 == 0, -1.0, 1.0))
    srv = p.Server(ctx, max_slots=4)
    for h in Hs + [quick]:   # every buffer of the requests below exists
        srv.sp2_server_wait(srv.sp2_server_submit(h, h.shape[0] // 2), h.shape[0], want_D=False)
    tk = [srv.sp2_server_submit(h, h.shape[0] // 2) for h in Hs]
    tq = srv.sp2_server_submit(quick, 320)
    _, _, st = srv.sp2_server_wait(tq, 640, want_D=False)
    running = []
    for t, h in zip(tk, Hs):
        try:
            srv.sp2_server_wait(t, h.shape[0], timeout_s=0.0, want_D=False)
            running.append(False)
        except p.Sp2Error as e:
            assert e.status == p.SP2_ETIMEOUT
            running.append(True)
    for t, h, r in zip(tk, Hs, running):
        if r:
            srv.sp2_server_wait(t, h.shape[0], want_D=False)
    srv.close()
    say(f"  quick one: {st['iterations']} products, {st['ms']:.1f} ms; others still running {running}")
    assert st["iterations"] < 16 and all(running)


@pytest.mark.parametrize("N", [2, 18, 19, 129])
def test_smallest_requests_equal_the_direct_solve(ctx, N):
    """Below N = 19 a request's row maxima take the place of its H check's
    partials, from there on they lie in D's memory with the partial sums: both
    ways two requests side by side equal the direct solve bit for bit."""
    import torch
    import paper_1203_6836_amd as p
    say(f"case served N={N}")
    rng = np.random.default_rng(N)
    Hs = []
    for _ in range(2):
        H = np.triu(rng.uniform(-0.3, 0.3, (N, N)) / np.sqrt(N), 1)
        Hs.append(H + H.T + np.diag(np.where(np.arange(N) % 2 == 0, -1.0, 1.0)))
    n_occ = (N + 1) // 2
    srv = p.Server(ctx, max_slots=2)
    tk = [srv.sp2_server_submit(H, n_occ) for H in Hs]
    out = [srv.sp2_server_wait(t, N) for t in tk]
    srv.close()
    for H, (D, _, st) in zip(Hs, out):
        Dd, sd = ctx.sp2_density_matrix(torch.from_numpy(H).cuda(), n_occ, p.options("int8x"))
        assert st["branches"] == sd["branches"]
        assert np.array_equal(D, Dd.cpu().numpy())
