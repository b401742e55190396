"""Large sparse problems on the entries that hold something or may come to: the bits of the sweeps over everything."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import drot_inputs

from . import parity_utils as pu

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _say(msg):
    print(f"[gpu-active] {msg}", flush=True)


@pytest.fixture(scope="module")
def drot():
    import paper_2305_18483_amd as drot_mod

    drot_mod.load_library()
    assert torch.cuda.is_available()
    return drot_mod


def _checks(solver):
    return [(c.iters, c.r_row, c.r_col) for c in solver.checks()]


def _both(drot, m, n, solve, launches=1, iterations=1, check_every=100):
    """solve(solver) -> tuple of arrays and numbers, with the default options and with every sweep in a launch of its own."""
    out = []
    for fused in (-1, 0):
        solver = drot.Solver(m, n, check_every=check_every)
        solver.set_fused_update(fused)
        out.append(solve(solver) + (_checks(solver),))
        accepted, refused, given_up = solver.cooperative_launches()
        assert refused == 0 and given_up == 0
        assert (accepted >= launches) if fused else accepted == 0, accepted
        runs = solver.active_runs()  # (an attempt whose entries do not fit is a launch as well)
        assert runs.launches == accepted and (runs.iterations >= iterations if fused else runs.iterations == 0), runs.iterations
        solver.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b) if isinstance(a, np.ndarray) else torch.equal(a, b) if torch.is_tensor(a) else a == b
    return out[0]


# 256-row groups and 256-column segments: one entry more than a whole number of them, and one less; fewer of either than there
# are rows and columns of workgroups; pairs forbidden, costs far above and below 1 (in few dimensions too many entries lie near the edge)
@pytest.mark.parametrize("m,n,kind,scale,forbid,d", [(3585, 3329, 1, 1.0, 0.0, 12), (3839, 4095, 0, 1.0, 0.3, 20), (2049, 5633, 1, 3.0e4, 0.0, 12),
                                                     (12289, 1000, 1, 1.0e-3, 0.1, 20)])
def test_active_entries_change_no_bit(drot, m, n, kind, scale, forbid, d):
    P = drot_inputs.with_entrywise_terms(drot_inputs.random_problem(m, n, seed=4100 + m, d=d, reg_kind=kind, lam=0.01), seed=4101, forbid_frac=forbid)
    P.C = (P.C * np.float32(scale)).astype(np.float32)

    def solve(solver):
        solver.set_skip_cost(0)
        res, X, phi, varphi = pu.gpu_solve(solver, P, 330, tol=1e-12, stepsize=float(P.rho) / scale)
        assert res.iters == 330
        return X, phi, varphi, res.objective, res.gap, res.r_row, res.r_col

    _say(f"stored cost {m}x{n}, kind {kind}, costs up to {scale:g}, forbidden {forbid:g}")
    _both(drot, m, n, solve, iterations=300)


# as many groups and segments as a workgroup holds, of both or of one, the last ones of one row and of one column; more blocks of
# eight rows and columns than waves to own them (32640 rows and columns), so that a wave owns two
@pytest.mark.parametrize("m,n", [(20225, 16641), (4097, 20480), (20480, 3073)])
def test_active_entries_of_the_largest_shapes_change_no_bit(drot, m, n):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(4150)
    xs, xt = torch.randn(m, 32, device=dev, generator=g), 0.3 + 1.4 * torch.randn(n, 32, device=dev, generator=g)
    C = torch.cdist(xs, xt) ** 2
    C /= C.max()
    p, q = (torch.rand(k, dtype=torch.float64, device=dev, generator=g) + 0.5 for k in (m, n))
    p, q = (p / p.sum()).float(), (q / q.sum()).float()

    def solve(solver):
        res = solver.solve(C, p, q, max_iters=150, tol=1e-12)
        return (res.X, *solver.duals(m, n, dev), res.objective, res.r_row, res.r_col)

    _say(f"stored cost {m}x{n}")
    _both(drot, m, n, solve, iterations=50)


# costs formed entry by entry as the sweeps' matrix instructions form them: more dimensions than one pass of theirs holds, points so small
# that products of their coordinates are denormal
@pytest.mark.parametrize("m,n,d,size", [(3585, 3329, 2, 1.0), (3400, 4097, 17, 1.0), (1200, 9729, 3, 1.0), (3585, 3329, 80, 1.0e-18),
                                        (1200, 9729, 201, 3.0e-19)])
def test_active_entries_of_point_clouds_change_no_bit(drot, m, n, d, size):
    P = drot_inputs.random_problem(m, n, seed=4200 + m, d=d, reg_kind=1, lam=0.001)
    dev = torch.device("cuda:0")
    xs, xt, p, q = (torch.from_numpy(a).to(dev) for a in ((P.xs * size).astype(np.float32), (P.xt * size).astype(np.float32), P.p, P.q))
    scale = 1.0 / float((torch.cdist(xs.double(), xt.double()) ** 2).max())

    def solve(solver):
        res = solver.solve_points(xs, xt, scale, p, q, reg_kind=1, lam=P.lam, max_iters=330, tol=1e-12)
        phi, varphi = solver.duals(m, n, dev)
        return res.X.cpu().numpy(), phi.cpu().numpy(), varphi.cpu().numpy(), res.objective, res.gap, res.r_row, res.r_col

    _say(f"point clouds {m}x{n}, d = {d}, of size {size:g}")
    _both(drot, m, n, solve, iterations=280 if d > 8 else 1)


def test_active_entries_across_calls_starts_and_stops(drot):
    m, n = 4000, 3900
    P = drot_inputs.random_problem(m, n, seed=4300, d=8, reg_kind=1, lam=0.01)
    dev = torch.device("cuda:0")
    C, p, q = (torch.from_numpy(a).to(dev) for a in (P.C, P.p, P.q))
    kw = dict(reg_kind=1, lam=P.lam)

    def continued(solver):  # calls that go on where the last one ended, one of them too short for a list of its own
        X = torch.empty(m, n, device=dev)
        out = []
        for k in (200, 5, 130, 16, 300):
            res = solver.solve(C, p, q, X_out=X, max_iters=k, tol=1e-12, **kw)
            solver.set_continue(True)
            out += [res.X.cpu().numpy(), res.objective, res.r_row]
        solver.set_continue(False)
        return tuple(out)

    _say("continued calls")
    cut = _both(drot, m, n, continued, launches=4, iterations=600, check_every=50)
    whole = _both(drot, m, n, lambda s: (s.solve(C, p, q, max_iters=651, tol=1e-12, **kw).X.cpu().numpy(),), iterations=600, check_every=50)
    assert np.array_equal(cut[-4], whole[0])

    def often(solver):  # 256 checks to a launch, and the next one goes on from there
        solver.set_skip_cost(0)
        return (solver.solve(C, p, q, max_iters=600, tol=1e-12, **kw).X.cpu().numpy(),)

    _both(drot, m, n, often, launches=2, iterations=580, check_every=2)

    def warm(solver):  # from potentials and a plan of another problem, then without a tolerance
        X = torch.from_numpy(whole[0]).to(dev) * 0.5
        res = solver.solve(C, p, q, X_out=X, phi0=torch.full((m,), 1e-5, device=dev), varphi0=torch.zeros(n, device=dev), max_iters=260, tol=1e-12, **kw)
        first = res.X.cpu().numpy()
        return first, solver.solve(C, p, q, max_iters=270, **kw).X.cpu().numpy()

    _say("warm start, no tolerance")
    _both(drot, m, n, warm, launches=2)

    probe = drot.Solver(m, n, check_every=10)
    probe.solve(C, p, q, max_iters=400, tol=1e-12, **kw)
    stop = max(probe.checks()[25].r_row, probe.checks()[25].r_col) * 1.0001

    def stopped(solver):  # at a check inside the launch, and on from there
        res = solver.solve(C, p, q, max_iters=4000, tol=stop, **kw)
        assert res.converged and 100 <= res.iters <= 260
        X, iters = res.X.cpu().numpy(), res.iters
        solver.set_continue(True)
        res = solver.solve(C, p, q, X_out=res.X, max_iters=150, tol=1e-12, **kw)
        return X, iters, res.X.cpu().numpy(), res.r_row

    _say(f"stops at a residual of {stop:.3e}")
    _both(drot, m, n, stopped, launches=2, check_every=10)


# calls that continue one another with the options that keep them off active entries in between, on a handle that holds the bounds of
# another problem: which launches record bounds by line, and which may read them, hangs on the options of each call
@pytest.mark.parametrize("off", ["gap_every", "fused_update", "screening", "gap_tolerance"])
@pytest.mark.parametrize("order", [(0, 1), (1, 0, 1)])
def test_active_entries_of_point_clouds_across_options(drot, off, order):
    m, n = 3585, 3329
    dev = torch.device("cuda:0")

    def points(seed):
        P = drot_inputs.random_problem(m, n, seed=seed, d=5)
        xs, xt, p, q = (torch.from_numpy(a).to(dev) for a in (P.xs.astype(np.float32), P.xt.astype(np.float32), P.p, P.q))
        return xs, xt, 1.0 / float((torch.cdist(xs, xt) ** 2).max()), p, q

    def switch(solver, on):
        if off == "gap_every":
            solver.set_gap_every(0 if on else 1)
        elif off == "fused_update":
            solver.set_fused_update(-1 if on else 0)
        elif off == "screening":
            solver.set_screening(-1 if on else 1)
        else:
            solver.set_gap_tolerance(0.0 if on else 1e-12)

    kw = dict(tol=1e-12)
    A, B = points(4500), points(4501)
    _say(f"point clouds, {off}, {order}")
    out = []
    for use in (True, False):
        solver = drot.Solver(m, n, check_every=20)
        solver.set_profile(not use)  # (every sweep in a launch of its own)
        solver.solve_points(*B, max_iters=200, **kw)
        taken, X = [], torch.empty(m, n, device=dev)
        for call, on in enumerate(order):
            solver.set_continue(call > 0)
            switch(solver, on)
            before = solver.cooperative_launches()[0]
            res = solver.solve_points(*A, X_out=X, max_iters=(200, 60, 120)[call], **kw)
            taken.append(solver.cooperative_launches()[0] - before)
        assert [t > 0 for t in taken] == [use and bool(on) for on in order], taken
        out.append((res.X.cpu().numpy(), *(v.cpu().numpy() for v in solver.duals(m, n, dev)), np.float64([res.objective, res.r_row, res.r_col])))
        solver.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("points", [False, True])
def test_a_launch_of_active_entries_that_gives_up_is_replaced_by_single_launches(drot, points):
    # one attempt per wait: every workgroup returns by itself.  A cold start comes out all the same, a warm one says that it has lost its point
    m, n = 3585, 3329
    dev = torch.device("cuda:0")
    P = drot_inputs.random_problem(m, n, seed=4600, d=5)
    C, xs, xt, p, q = (torch.from_numpy(a).to(dev) for a in (P.C, P.xs.astype(np.float32), P.xt.astype(np.float32), P.p, P.q))
    scale = 1.0 / float((torch.cdist(xs, xt) ** 2).max())
    kw = dict(max_iters=200, tol=1e-12)

    def solve(solver, **more):
        return solver.solve_points(xs, xt, scale, p, q, **kw, **more) if points else solver.solve(C, p, q, **kw, **more)

    def state(solver, res):
        return res.X.clone(), *solver.duals(m, n, dev), res.objective, res.r_row, _checks(solver)

    single, solver = drot.Solver(m, n), drot.Solver(m, n)
    single.set_fused_update(0)
    ref = state(single, solve(single))
    _say(f"a launch that gives up, points {points}")
    solver.set_grid_polls(1)
    for _ in range(2):
        got = state(solver, solve(solver))
        assert all(torch.equal(a, b) if torch.is_tensor(a) else a == b for a, b in zip(got, ref))
        assert solver.cooperative_launches() == (1, 0, 1)
    solver = drot.Solver(m, n)
    solver.set_grid_polls(1)
    with pytest.raises(drot.DrotError) as e:
        solve(solver, X_out=ref[0].clone(), phi0=ref[1], varphi0=ref[2])
    assert e.value.code == drot.binding.DROT_ERR_HIP and solver.cooperative_launches() == (1, 0, 1)


_REFUSED = '''
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # first, so that its symbol is found before the runtime's own
import numpy as np, torch
import drot_inputs
import paper_2305_18483_amd as drot
m, n = 3585, 3329
dev = torch.device("cuda:0")
P = drot_inputs.random_problem(m, n, seed=4700, d=12)
C, xs, xt, p, q = (torch.from_numpy(a).to(dev) for a in (P.C, P.xs.astype(np.float32), P.xt.astype(np.float32), P.p, P.q))
scale = 1.0 / float((torch.cdist(xs, xt) ** 2).max())
for points in (False, True):
    out = []
    for single in (False, True):
        solver = drot.Solver(m, n)
        if single:
            solver.set_fused_update(0)
        before = shim.refusals()
        for _ in range(2):  # (the handle asks once)
            kw = dict(max_iters=200, tol=1e-12)
            res = solver.solve_points(xs, xt, scale, p, q, **kw) if points else solver.solve(C, p, q, **kw)
            out.append((res.X.clone(), *solver.duals(m, n, dev), res.objective, res.r_row))
        assert shim.refusals() - before == solver.cooperative_launches()[1] == (0 if single else 1)
        assert solver.cooperative_launches()[0] == solver.active_runs().launches == 0
    for got in out[:-1]:
        assert all(torch.equal(a, b) if torch.is_tensor(a) else a == b for a, b in zip(got, out[-1]))
print("refused and done", shim.refusals(), flush=True)
'''


def test_a_launch_of_active_entries_that_is_refused_is_replaced_by_single_launches(tmp_path):
    # a function of the same name, loaded ahead of the runtime in a child process, accepts no cooperative launch
    src, lib = tmp_path / "refuse.cpp", tmp_path / "librefuse.so"
    src.write_text('''
struct dim3 { unsigned x, y, z; };
static int refused;
extern "C" int refusals() { return refused; }
extern "C" int hipLaunchCooperativeKernel(const void*, dim3, dim3, void**, unsigned, void*) {
  ++refused;
  return 720;  // hipErrorCooperativeLaunchTooLarge
}
''')
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    _say("refused launches, in a child process")
    env = dict(os.environ, PYTHONPATH=os.pathsep.join(x for x in (ROOT, os.environ.get("PYTHONPATH")) if x))
    proc = subprocess.run([sys.executable, "-c", _REFUSED, str(lib)], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                          timeout=100, env=env)
    assert proc.returncode == 0 and "refused and done 2" in proc.stdout, proc.stdout


# launches that end early: entries that do not fit at the first list (misfits), and later on (outgrown: X goes back to what it was before an
# iteration that nobody counts, in the workgroups that have lists)
@pytest.mark.parametrize("points,d,lam,ended", [(False, 2, 0.0, "misfits"), (False, 5, 0.0, "outgrown"), (False, 5, 100.0, "outgrown"), (True, 1, 0.0, "misfits"),
                                                (True, 2, 100.0, "outgrown")])
def test_active_entries_that_do_not_fit_leave_the_solve_to_the_sweeps(drot, points, d, lam, ended):
    m, n = 3585, 3329
    P = drot_inputs.random_problem(m, n, seed=4400, d=d, reg_kind=1 if lam else 0, lam=lam)
    dev = torch.device("cuda:0")
    C, xs, xt, p, q = (torch.from_numpy(a).to(dev) for a in (P.C, P.xs.astype(np.float32), P.xt.astype(np.float32), P.p, P.q))
    scale = 1.0 / float((torch.cdist(xs, xt) ** 2).max())
    kw = dict(reg_kind=1 if lam else 0, lam=lam, max_iters=420, tol=1e-12)

    def solve(solver):
        solver.set_skip_cost(0)
        res = solver.solve_points(xs, xt, scale, p, q, **kw) if points else solver.solve(C, p, q, **kw)
        if solver.cooperative_launches()[0]:
            runs = solver.active_runs()
            assert (runs.misfits, runs.outgrown) == ((1, 0) if ended == "misfits" else (0, 1)), (runs.misfits, runs.outgrown)
        return (res.X.cpu().numpy(), *(v.cpu().numpy() for v in solver.duals(m, n, dev)), res.objective, res.r_row)

    _say(f"entries that do not fit, points {points}, d = {d}, lam = {lam:g}")
    _both(drot, m, n, solve, iterations=1 if ended == "outgrown" else 0)


def test_a_band_of_entries_leaves_the_solve_to_the_sweeps(drot):
    # row i holds its mass near column i: the workgroups on the diagonal of 16 x 16 have sixteen times their part of the entries, and
    # a quadratic term of middling strength keeps dozens of them in every row
    m = n = 6000
    x = np.linspace(0.0, 1.0, m, dtype=np.float32)
    P = drot_inputs.random_problem(m, n, seed=4400, d=2, reg_kind=1, lam=6.0)
    P.C = np.ascontiguousarray((x[:, None] - x[None, :]) ** 2)
    dev = torch.device("cuda:0")
    C, p, q = (torch.from_numpy(a).to(dev) for a in (P.C, P.p, P.q))

    def solve(solver):
        solver.set_skip_cost(0)
        res = solver.solve(C, p, q, reg_kind=1, lam=6.0, max_iters=420, tol=1e-12)
        return res.X.cpu().numpy(), res.objective, res.r_row

    _say("a band of entries")
    X = _both(drot, m, n, solve)[0]
    assert (X > 0).sum() > m
