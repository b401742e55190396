"""Launches whose workgroups wait for one another, where they are refused or give up: the solves come out by single launches.

The child processes come first: a system may let only one process at a time launch that way, and this one has done so once a
solve has run in it.
"""
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
    print(f"[gpu-cooperative] {msg}", flush=True)


def _child_env():
    return dict(os.environ, PYTHONPATH=os.pathsep.join(x for x in (ROOT, os.environ.get("PYTHONPATH")) if x))


@pytest.fixture(scope="module")
def drot():
    import paper_2305_18483_amd as drot_mod

    drot_mod.load_library()
    assert torch.cuda.is_available()
    return drot_mod


_REFUSED = '''
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # first, so that its symbol is found before the runtime's own
import numpy as np, torch
import drot_inputs
import paper_2305_18483_amd as drot
dev = torch.device("cuda:0")
for m, n in ((600, 1024), (2300, 2528)):
    P = drot_inputs.random_problem(m, n, seed=2660 + m, reg_kind=1, lam=0.3)
    C, p, q = (torch.from_numpy(a).to(dev) for a in (P.C, P.p, P.q))
    kw = dict(reg_kind=1, lam=P.lam, max_iters=130, tol=1e-12)
    solver = drot.Solver(m, n)
    before = shim.refusals()
    X = solver.solve(C, p, q, **kw).X.clone()
    assert shim.refusals() == before + 1, "the handle asked again"
    again = solver.solve(C, p, q, **kw).X.clone()
    assert shim.refusals() == before + 1
    single = drot.Solver(m, n)
    single.set_profile(True)
    ref = single.solve(C, p, q, **kw).X
    assert torch.equal(X, ref) and torch.equal(again, ref)
    assert solver.cooperative_launches() == (0, 1, 0) and single.cooperative_launches() == (0, 0, 0)
    Xs = torch.empty_like(C)
    info = torch.zeros(64, dtype=torch.uint8, device=dev)
    drot.solve_static(C, p, q, Xs, info_out=info, **kw)
    torch.cuda.synchronize()
    assert drot.read_info(info).iters == 130 and torch.equal(Xs, ref) and shim.refusals() == before + 2
print("refused and done", shim.refusals(), flush=True)

# let through, with one attempt per wait in place of 2^25: the static entry point, whose caller may not read the info block,
# leaves no plan that could be taken for one
(path,) = {line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line}
real = ctypes.cast(ctypes.CDLL(path).hipLaunchCooperativeKernel, ctypes.c_void_p)
shim.let_through(real, 1 << 25, 1)
phi, varphi = torch.zeros(m, device=dev), torch.zeros(n, device=dev)
drot.solve_static(C[:1024], p[:1024].contiguous(), q, Xs[:1024], phi_out=phi[:1024], varphi_out=varphi, info_out=info, **kw)
torch.cuda.synchronize()
assert shim.lowered() == (1 if shim.failed() else 2)
if shim.failed():  # (the system lets one process at a time launch that way: the caller's, where it has done so before)
    print("gave up True 0.0: not tried", flush=True)
else:
    try:
        drot.read_info(info)
    except drot.DrotError:
        print("gave up", bool(torch.isnan(Xs[:1024]).all() and torch.isnan(phi[:1024]).all() and torch.isnan(varphi).all()),
              float(phi[1024:].abs().max()), flush=True)

# "not for this process" (hipErrorIllegalState): one that asks is enough
shim.refuse_with(401)
before = shim.refusals()
single.set_profile(False)
for solver in (single, drot.Solver(m, n), drot.Solver(m, n)):
    assert torch.equal(solver.solve(C, p, q, **kw).X, ref)
drot.solve_static(C, p, q, Xs, **kw)
torch.cuda.synchronize()
assert torch.equal(Xs, ref)
print("asked", shim.refusals() - before if not shim.failed() else 1, flush=True)
'''


def test_a_launch_that_is_refused_is_replaced_by_single_launches(tmp_path):
    # a runtime that accepts no cooperative launch (as for a process that may not use every compute unit): a function of
    # the same name, loaded ahead of the runtime in a child process, refuses them all
    src = tmp_path / "refuse.cpp"
    src.write_text('''
struct dim3 { unsigned x, y, z; };
typedef int (*launch_t)(const void*, dim3, dim3, void**, unsigned, void*);
static int refused, lowered_, failed_, from, to, code = 720;  // hipErrorCooperativeLaunchTooLarge
static launch_t real;
extern "C" int refusals() { return refused; }
extern "C" int lowered() { return lowered_; }
extern "C" int failed() { return failed_; }
extern "C" void refuse_with(int error) { real = 0; code = error; }
extern "C" void let_through(void* f, int was, int now) { real = (launch_t)f; from = was; to = now; }
extern "C" int hipLaunchCooperativeKernel(const void* f, dim3 grid, dim3 block, void** args, unsigned lds, void* stream) {
  if (!real) {
    ++refused;
    return code;
  }
  // (the one argument, a struct of some 270 bytes that ends in: iterations, 0 or 1, a small number, attempts per wait)
  for (int* w = (int*)args[0]; w < (int*)args[0] + 64; ++w)
    if (w[0] >= 4 && w[0] <= 100 && (w[1] == 0 || w[1] == 1) && w[2] >= 1 && w[2] < 1000 && w[3] == from) {
      w[3] = to;
      ++lowered_;
      break;
    }
  const int rc = real(f, grid, block, args, lds, stream);
  if (rc) failed_ = rc;
  return rc;
}
''')
    lib = tmp_path / "librefuse.so"
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    _say("refused launches, in a child process")
    proc = subprocess.run([sys.executable, "-c", _REFUSED, str(lib)], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                          text=True, timeout=100, env=_child_env())
    assert proc.returncode == 0 and "refused and done 4" in proc.stdout and "gave up True 0.0" in proc.stdout and "asked 1" in proc.stdout, proc.stdout


_SECOND = '''
import sys
import numpy as np, torch
import drot_inputs
import paper_2305_18483_amd as drot
dev = torch.device("cuda:0")
P = drot_inputs.random_problem(900, 1000, seed=2670, reg_kind=1, lam=0.3)
C, p, q = (torch.from_numpy(a).to(dev) for a in (P.C, P.p, P.q))
X = drot.Solver(900, 1000).solve(C, p, q, reg_kind=1, lam=P.lam, max_iters=130).X
np.save(sys.argv[1], X.cpu().numpy())
'''


def test_a_second_process_on_the_gpu(drot, tmp_path):
    # this process has launched that way, and stays: the second one may be refused (it was, with an error as the result)
    P = drot_inputs.random_problem(900, 1000, seed=2670, reg_kind=1, lam=0.3)
    _say("a second process")
    solver = drot.Solver(P.m, P.n)
    _, X, _, _ = pu.gpu_solve(solver, P, 130)
    pu.assert_held_on_the_chip(solver)
    out = tmp_path / "second.npy"
    proc = subprocess.run([sys.executable, "-c", _SECOND, str(out)], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                          text=True, timeout=100, env=_child_env())
    assert proc.returncode == 0, proc.stdout
    assert np.array_equal(np.load(out), X)


@pytest.mark.parametrize("m,n", [(1000, 1000), (2300, 2500)])
def test_a_launch_that_gives_up_is_replaced_by_single_launches(drot, m, n):
    # one attempt per wait: the first word that is still on its way ends the launch (every workgroup returns by itself).  A
    # cold start comes out all the same, with the bits of single launches; a warm start says that it has lost its point; the
    # handle goes on without such launches
    P = drot_inputs.random_problem(m, n, seed=2650 + m, reg_kind=1, lam=0.3)
    C, p, q, _ = pu.to_dev(P)
    _say(f"a launch that gives up, {m}x{n}")
    _, X_ref, phi_ref, varphi_ref = pu.gpu_solve(drot.Solver(m, n), P, 150, tol=1e-12)
    solver = drot.Solver(m, n)
    solver.set_grid_polls(1)
    for _ in range(2):
        res, X, phi, varphi = pu.gpu_solve(solver, P, 150, tol=1e-12)
        assert res.iters == 150 and [c.iters for c in solver.checks()] == [100, 150]
        assert np.array_equal(X, X_ref) and np.array_equal(phi, phi_ref) and np.array_equal(varphi, varphi_ref)
    pu.assert_held_on_the_chip(solver, given_up=1)
    solver = drot.Solver(m, n)
    solver.set_grid_polls(1)
    phi0, varphi0 = torch.zeros(m, device=C.device), torch.zeros(n, device=C.device)
    kw = dict(reg_kind=1, lam=P.lam, max_iters=60, phi0=phi0, varphi0=varphi0)
    with pytest.raises(drot.DrotError) as e:
        solver.solve(C, p, q, X_out=torch.zeros_like(C), **kw)
    assert e.value.code == drot.binding.DROT_ERR_HIP
    assert solver.cooperative_launches() == (1, 0, 1)
    again = solver.solve(C, p, q, X_out=torch.zeros_like(C), **kw).X
    assert torch.equal(again, drot.Solver(m, n).solve(C, p, q, X_out=torch.zeros_like(C), **kw).X)
    for bad in (0, -1, (1 << 30) + 1):
        with pytest.raises(drot.DrotError):
            solver.set_grid_polls(bad)


def test_a_launch_of_slabs_that_gives_up_is_replaced_by_single_launches(drot):
    P = drot_inputs.random_problem(1500, 1000, seed=2655, reg_kind=2, lam=0.1, mu=0.02, num_classes=2)
    _say("a launch of slabs that gives up")
    _, X_ref, phi_ref, varphi_ref = pu.gpu_solve(drot.Solver(P.m, P.n), P, 150, tol=1e-12)
    solver = drot.Solver(P.m, P.n)
    solver.set_grid_polls(1)
    for _ in range(2):
        res, X, phi, varphi = pu.gpu_solve(solver, P, 150, tol=1e-12)
        assert res.iters == 150 and [c.iters for c in solver.checks()] == [100, 150]
        assert np.array_equal(X, X_ref) and np.array_equal(phi, phi_ref) and np.array_equal(varphi, varphi_ref)
    pu.assert_held_on_the_chip(solver, given_up=1)
