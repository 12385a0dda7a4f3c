"""Resident sweeps (a chunk of sweeps in one launch) against the two-sweep launches and the
oracle (needs an MI355X).

Both forms compute a cell's update with the same operations in the same order, so their states
are equal bit for bit after an even number of sweeps (an odd remainder of the two-sweep launches
is a single sweep of other arithmetic); the oracle bound is that of the other FP32 forms (1e-5 after 401 updates,
see test_gpu_fp32_parity).  Boxes cover every column length, one workgroup and many, ragged
sub-boxes in x, y and z, a top plane of one cell, and chunks of two to 401 sweeps.
"""
import threading
import time
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

from paper_2502_08034_amd import inputs as I

pytestmark = pytest.mark.gpu

FINITE = dict(s_in=1.0, s_eq=0.0, Da=0.45, mode=0)
PINNED = dict(s_in=0.0, s_eq=1.0, Da=0.0, mode=1)


@pytest.fixture(scope="module")
def sv():
    from paper_2502_08034_amd import socfv
    assert torch.cuda.is_available()
    return socfv


def inputs_of(shape, kappa=False):
    nx, ny, nz = shape
    if min(ny, nz) < 12:                         # plain channel
        solid, u = I.plug_flow_case(nx, ny, nz, 0.7)
    else:
        solid = I.fibres_nonoverlap(nx, ny, nz, 2.5, 0.88, 7).solid
        u = I.darcy_velocity(solid, 1.0, device="cuda", as_numpy=False)
    return solid, u, I.lognormal_activity(solid, 0.3, seed=9) if kappa else None


def problem(sv, inputs):
    solid, u, k = inputs
    return sv.Problem.create(solid, *u, kappa=k)


def both(sv, pb, **kw):
    """The resident launches' state and the two-sweep launches' (and their statistics)."""
    p = sv.params(precision="fp32", **kw)
    out = [sv.solve_soc_steady(pb.ctx, p)]
    if kw["mode"] == 0:
        out.append(sv.solve_soc_adjoint(pb.ctx, p, want_psi=True)[2:])
    sv.set_tiles(pb.ctx, 0, 0, 0, 1)
    out.append(sv.solve_soc_steady(pb.ctx, p))
    if kw["mode"] == 0:
        out.append(sv.solve_soc_adjoint(pb.ctx, p, want_psi=True)[2:])
    return out


@pytest.mark.parametrize("shape,kappa,mode", [
    ((1, 1, 1), False, FINITE), ((33, 3, 2), False, FINITE), ((600, 3, 2), True, FINITE),
    ((5, 600, 7), False, FINITE), ((7, 5, 901), False, FINITE),         # few columns, long ones
    ((64, 32, 33), False, PINNED), ((131, 33, 41), True, FINITE),       # 4 cells a column
    ((129, 63, 65), False, FINITE),                                     # 8
    ((175, 89, 89), False, PINNED),                                     # 12
    ((191, 97, 95), True, FINITE),                                      # 16
    ((253, 97, 99), False, FINITE),                                     # 20
    ((256, 120, 118), False, PINNED), ((256, 128, 128), False, FINITE),  # lean columns
    ((256, 128, 127), False, PINNED),
])
def test_resident_sweeps_equal_the_two_sweep_launches(sv, shape, kappa, mode):
    inputs = inputs_of(shape, kappa)
    for check, sweeps in ((200, 400), (2, 6), (30, 70)):
        runs = both(sv, problem(sv, inputs), tol=0.0, max_iter=sweeps, check_every=check, **mode)
        half = len(runs) // 2
        for a, b in zip(runs[:half], runs[half:]):
            assert a[1].iterations == b[1].iterations == sweeps
            assert torch.equal(a[0], b[0]), (shape, check, sweeps)


@pytest.mark.parametrize("mode", [FINITE, PINNED])
def test_resident_sweeps_match_the_oracle(sv, orc, mode):
    inputs = inputs_of((67, 35, 29))
    pb, solid, u = problem(sv, inputs), inputs[0], inputs[1]
    u = [np.asarray(v.cpu() if isinstance(v, torch.Tensor) else v) for v in u]
    op = orc.Problem(solid, *u, s_in=mode["s_in"], s_eq=mode["s_eq"], Da=mode["Da"],
                     pinned=bool(mode["mode"]))
    s0 = op.initial_state()
    r0, _ = orc.residual(op, s0)
    ref = s0 + orc.correction_iterate(op, r0, 0.4 / orc.max_diag(op), 401)
    s, st = sv.solve_soc_steady(pb.ctx, sv.params(precision="fp32", tol=0.0, max_iter=401,
                                                  check_every=401, **mode))
    assert st.iterations == 401
    assert np.abs(s.cpu().numpy() - ref)[solid == 0].max() <= 1e-5


def test_a_launch_that_is_given_up_loses_nothing(sv):
    # wait limit 0: every resident launch is given up at its first missing value, and the solve
    # and the adjoint go on with the two-sweep launches from the untouched input; the FP32 sweeps
    # are the same bit for bit, the 100 FP64 sweeps of the polish to their rounding
    inputs = inputs_of((96, 48, 40))
    ref, pb = problem(sv, inputs), problem(sv, inputs)
    sv.set_wait_limit(pb.ctx, 0.0)
    with pytest.raises(sv.SocfvError):
        sv.set_wait_limit(pb.ctx, -1.0)
    p = sv.params(precision="fp32", tol=1e-8, check_every=100, **FINITE)
    for _ in range(2):
        (s, st), (r, rt) = sv.solve_soc_steady(pb.ctx, p), sv.solve_soc_steady(ref.ctx, p)
        assert st.status == sv.OK and st.iterations == rt.iterations
        assert (s - r).abs().max() <= 1e-12
        ga, gb = sv.solve_soc_adjoint(pb.ctx, p), sv.solve_soc_adjoint(ref.ctx, p)
        assert ga[3].iterations == gb[3].iterations
        assert (ga[0] - gb[0]).abs().max() <= 1e-11 * gb[0].abs().max()


@pytest.mark.parametrize("shape,threads", [((64, 32, 33), 6), ((175, 89, 89), 3)])
def test_solves_of_several_threads_wait_for_their_turn(sv, shape, threads):
    # launches that do not fit the chip together are ordered one behind the other: none runs into
    # the time limit (1 s a launch; all the solves take less), and the results are a single
    # thread's
    inputs = inputs_of(shape)
    ref = problem(sv, inputs)
    p = sv.params(precision="fp32", tol=0.0, max_iter=2000, check_every=20, **FINITE)
    s0, _ = sv.solve_soc_steady(ref.ctx, p)
    pbs = [problem(sv, inputs) for _ in range(threads)]
    start = threading.Barrier(threads)

    def run(pb):
        start.wait()
        return [sv.solve_soc_steady(pb.ctx, p)[0] for _ in range(3)]

    t0 = time.perf_counter()
    with ThreadPoolExecutor(threads) as pool:
        out = list(pool.map(run, pbs))
    assert time.perf_counter() - t0 < 1.0
    assert all(torch.equal(s, s0) for runs in out for s in runs)


@pytest.mark.parametrize("shape,kappa,mode", [
    ((33, 3, 2), False, FINITE), ((64, 32, 33), True, FINITE), ((129, 63, 65), False, PINNED),
    ((175, 89, 89), True, FINITE),                                      # lean columns
    ((191, 97, 95), False, PINNED),
])
def test_resident_fp64_sweeps_equal_the_march(sv, shape, kappa, mode):
    # the same update with the terms summed in another order: 300 non-expansive updates round
    # about ten operations each, 1e-16 relative to |s| <= 1 (psi: to its largest value)
    inputs = inputs_of(shape, kappa)
    pb = problem(sv, inputs)
    p = sv.params(precision="fp64", tol=0.0, max_iter=301, check_every=100, **mode)
    runs = []
    for _ in range(2):
        s, st = sv.solve_soc_steady(pb.ctx, p)
        psi = sv.solve_soc_adjoint(pb.ctx, p, want_psi=True)[2] if mode is FINITE else s
        runs.append((s, psi, st))
        sv.set_tiles(pb.ctx, 0, 0, 0, 1)
    (s1, a1, r1), (s2, a2, r2) = runs
    assert r1.iterations == r2.iterations == 301
    assert (s1 - s2).abs().max() <= 1e-12
    assert (a1 - a2).abs().max() <= 1e-12 * a2.abs().max()
    assert abs(r1.residual - r2.residual) <= 1e-9 * r2.residual


def batch_of(sv, shapes):
    return [problem(sv, inputs_of(shape, kappa)) for shape, kappa in shapes]


BATCH = [((64, 32, 33), False), ((131, 33, 41), True), ((129, 63, 65), False),
         ((45, 20, 17), False), ((96, 80, 77), True)]


def test_batched_resident_sweeps_equal_the_single_solves(sv):
    # problems with and without an activity field, finite and pinned, one with a cap on its
    # sweeps: the same states as alone (the FP32 sweeps bit for bit, the polish to its rounding)
    pbs = batch_of(sv, BATCH)
    ps = [sv.params(precision="fp32", tol=1e-9, **(PINNED if k == 2 else FINITE))
          for k in range(len(pbs))]
    ps[3].max_iter = 600
    states, stats = sv.batch_solve([pb.ctx for pb in pbs], ps)
    for k, (pb, p, s, st) in enumerate(zip(pbs, ps, states, stats)):
        r, rt = sv.solve_soc_steady(pb.ctx, p)
        assert st.status == rt.status == (sv.NOT_CONVERGED if k == 3 else sv.OK), k
        assert st.iterations == rt.iterations and st.cycles == rt.cycles, k
        assert (s - r).abs().max() <= 1e-12, k


def test_a_batch_beyond_the_chip_runs_in_turns(sv):
    # more cells than the chip holds at once (four boxes of 1.4 million)
    inputs = inputs_of((175, 89, 89))
    pbs = [problem(sv, inputs) for _ in range(4)]
    p = sv.params(precision="fp32", tol=1e-6, **FINITE)
    states, stats = sv.batch_solve([pb.ctx for pb in pbs], [p] * 4)
    s, st = sv.solve_soc_steady(pbs[0].ctx, p)
    for x, xt in zip(states, stats):
        assert xt.status == sv.OK and xt.iterations == st.iterations
        assert (x - s).abs().max() <= 1e-12


def test_a_batch_whose_launches_are_given_up_still_converges(sv):
    # wait limit 0 on two of the problems: they go on in the tiled launches, from a state that
    # the correction so far has gone into; the fixed point is the same
    pbs = batch_of(sv, BATCH)
    p = [sv.params(precision="fp32", tol=1e-9, **FINITE) for _ in pbs]
    for k in (0, 4):
        sv.set_wait_limit(pbs[k].ctx, 0.0)
    states, stats = sv.batch_solve([pb.ctx for pb in pbs], p)
    for pb, q, s, st in zip(pbs, p, states, stats):
        assert st.status == sv.OK and st.residual < 1e-9
        r, _ = sv.solve_soc_steady(pb.ctx, q)
        assert (s - r).abs().max() <= 1e-7          # both within the tolerance of the fixed point


@pytest.mark.parametrize("shape,kappa", [((33, 3, 2), False), ((64, 32, 33), True),
                                         ((129, 63, 65), False), ((150, 80, 81), True)])
def test_resident_nernst_equals_the_launches(sv, shape, kappa):
    # the same iteration with the transport rate's terms summed in another order (1e-16 of |s|
    # <= 1); the overpotential divides it by a k0 sqrt(s (1 - s)) of order one and relaxes
    inputs = inputs_of(shape, kappa)
    pb = problem(sv, inputs)
    p = sv.params(tol=0.0, max_iter=301, check_every=100, s_in=0.2, s_eq=0.7, Da=5.0, mode=0)
    runs = []
    for _ in range(2):
        runs.append(sv.solve_nernst(pb.ctx, p, omega=0.3, want_eta=True))
        sv.set_tiles(pb.ctx, 0, 0, 0, 1)
    (s1, e1, r1), (s2, e2, r2) = runs
    assert r1.iterations == r2.iterations == 301
    assert (s1 - s2).abs().max() <= 1e-12 and (e1 - e2).abs().max() <= 1e-11
    assert abs(r1.residual - r2.residual) <= 1e-9 * max(r2.residual, 1e-12)
    sv.set_tiles(pb.ctx, 0, 0, 0, 1)
    fresh = problem(sv, inputs)
    sv.set_wait_limit(fresh.ctx, 0.0)            # given up: the launches go on
    s3, e3, _ = sv.solve_nernst(fresh.ctx, p, omega=0.3, want_eta=True)
    assert (s3 - s2).abs().max() <= 1e-12 and (e3 - e2).abs().max() <= 1e-11


def test_given_up_launches_of_one_kind_leave_the_others(sv):
    # an FP32 solve, an FP64 solve, an adjoint and a Nernst solve on one context, each given up
    # once (the flag that says so is cleared by whoever finds it), then all four again with the
    # ordinary limit: the results of a context on which nothing was given up, to the FP64 sweeps'
    # rounding
    inputs = inputs_of((96, 48, 40))
    ref, pb = problem(sv, inputs), problem(sv, inputs)
    kw = dict(tol=0.0, max_iter=300, check_every=100)
    p32, p64 = (sv.params(precision=v, **kw, **FINITE) for v in ("fp32", "fp64"))
    pn = sv.params(s_in=0.2, s_eq=0.7, Da=5.0, mode=0, **kw)

    def kinds(ctx):
        yield sv.solve_soc_steady(ctx, p32)[0]
        yield sv.solve_soc_steady(ctx, p64)[0]
        yield sv.solve_soc_adjoint(ctx, p64, want_psi=True)[2]
        yield sv.solve_nernst(ctx, pn, omega=0.3)[0]

    want = list(kinds(ref.ctx))
    for limit in (0.0, 1.0):
        sv.set_wait_limit(pb.ctx, limit)
        for k, (a, b) in enumerate(zip(kinds(pb.ctx), want)):
            assert (a - b).abs().max() <= 1e-12 * max(1.0, float(b.abs().max())), (limit, k)


@pytest.mark.parametrize("shape", [(64, 32, 33), (175, 89, 89)])
@pytest.mark.parametrize("check", [2, 4, 6, 8])
def test_chunks_around_the_fewest_sweeps_of_a_resident_launch(sv, shape, check):
    # chunks below and above it, and solves whose last chunk is shorter than the others: FP32 states
    # equal bit for bit, FP64 and Nernst ones to their rounding
    inputs = inputs_of(shape)
    for sweeps in (3 * check, 2 * check + 2):
        kw = dict(tol=0.0, max_iter=sweeps, check_every=check)
        pb, res = problem(sv, inputs), []
        p64, pn = sv.params(precision="fp64", **kw, **FINITE), sv.params(
            s_in=0.2, s_eq=0.7, Da=5.0, mode=0, **kw)
        runs = both(sv, problem(sv, inputs), **kw, **FINITE)
        for a, b in zip(runs[:2], runs[2:]):
            assert a[1].iterations == b[1].iterations == sweeps
            assert torch.equal(a[0], b[0])
        for _ in range(2):
            res.append([sv.solve_soc_steady(pb.ctx, p64)[0],
                        sv.solve_soc_adjoint(pb.ctx, p64, want_psi=True)[2],
                        sv.solve_nernst(pb.ctx, pn, omega=0.3)[0]])
            sv.set_tiles(pb.ctx, 0, 0, 0, 1)
        for a, b in zip(*res):
            assert (a - b).abs().max() <= 1e-12 * max(1.0, float(b.abs().max()))


@pytest.mark.parametrize("shape", [(96, 48, 40), (258, 128, 130)])     # fits the chip / does not
def test_autotune_leaves_the_results(sv, shape):
    # it times shapes of the launches that boxes beyond the chip take and keeps the fastest; a
    # box that fits goes on with its resident launches
    pb = problem(sv, inputs_of(shape))
    p = sv.params(precision="fp32", tol=0.0, max_iter=80, check_every=40, **FINITE)
    s, st = sv.solve_soc_steady(pb.ctx, p)
    ty, zc, zc2 = sv.autotune(pb.ctx, 4)
    assert ty in (1, 2, 4, 8, 16) and 1 <= zc <= 64 and 1 <= zc2 <= 128
    t, tt = sv.solve_soc_steady(pb.ctx, p)
    assert tt.iterations == st.iterations == 80 and (tt.tile_y, tt.z_chunk) == (ty, zc)
    assert torch.equal(s, t)


WORKER = """
import sys, time
sys.path.insert(0, sys.argv[1])
import torch
from paper_2502_08034_amd import inputs as I, socfv as sv
boxes = [(64, 32, 32), (175, 89, 89), (128, 64, 64), (96, 48, 48)]
kw = dict(tol=0.0, max_iter=1000, check_every=200, s_in=1.0, s_eq=0.0, Da=0.45, mode=0)
worst, sums = 0.0, {}
for k in range(-4, 40):
    solid, u = I.plug_flow_case(*boxes[(k + int(sys.argv[2])) % 4], 0.7)
    pb = sv.Problem.create(solid, *u)
    t = time.perf_counter()
    s, st = sv.solve_soc_steady(pb.ctx, sv.params(precision="fp32", **kw))
    r, _ = sv.solve_soc_steady(pb.ctx, sv.params(precision="fp64", **kw))
    ux = sv.solve_stokes(pb.ctx, cfl=3.0, max_steps=20, tol=0.0)[0]
    torch.cuda.synchronize()
    if k >= 0:                                   # (the first ones load the kernels)
        worst = max(worst, time.perf_counter() - t)
    got = [float(v.double().sum()) for v in (s, r, ux)]
    want = sums.setdefault(solid.shape, got)
    assert st.iterations == 1000
    assert got[0] == want[0] and abs(got[1] - want[1]) <= 1e-12 * abs(want[1]) and got[2] == want[2]
print(worst)
"""


def test_processes_that_share_the_gpu_make_headway(sv):
    # launches of several processes can each hold a part of the CUs and wait for the rest: they give
    # up soon, do some chunks otherwise and try again.  Without contention the three calls take 0.02
    # to 0.07 s; a launch that waits a second, or a context that then stays with the slow launches,
    # would show.  The results are the same
    import subprocess
    import sys
    import os
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    procs = [subprocess.Popen([sys.executable, "-c", WORKER, root, str(k)], stdout=subprocess.PIPE,
                              text=True) for k in range(3)]
    try:
        out = [p.communicate(timeout=100)[0] for p in procs]
    finally:
        for p in procs:
            p.kill()
    assert all(p.returncode == 0 for p in procs)
    assert all(float(o) < 0.7 for o in out), out
