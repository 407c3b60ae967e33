"""The resident pressure CG (a whole Jacobi solve in one launch) against the
oracle, at the edges of its parts (4096 cells), of its groups (32 parts) and
of its slot counts, and where its waits between workgroups run out.

Tolerance: both sides take the same iteration counts and differ only in the
order of FP64 sums, so the FP64 parity bound of 1e-9 (relative L2) applies.
"""
import ctypes as ct
import sys
import threading

import numpy as np
import pytest

from oracle import oracle as orc
from paper_1207_1571_amd import meshgen as mg
from paper_1207_1571_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-9


def _case(shape, perm=None, kind="cavity", jitter=0.0):
    if kind == "duct":
        c = wl.duct(shape, Re=50.0, jitter=jitter, jitter_seed=3, mode="piso", dt=0.01)
        return c if perm is None else c.with_(mesh=mg.random_permutation(c.mesh, perm))
    return wl.cavity(shape, Re=100.0, dt=0.01, perm_seed=perm, jitter=jitter, jitter_seed=3)


def _inputs(mesh, seed):
    rng = np.random.default_rng(seed)
    rhs = rng.normal(size=mesh.n_cells)
    return rng.uniform(0.5, 2.0, mesh.n_faces), rhs - rhs.mean(), rng.normal(size=mesh.n_cells) * 0.1


def _solve(c, inputs, tol, max_iter, stream=None):
    import torch
    g, r, p = (torch.from_numpy(a.copy()).cuda() for a in inputs)
    torch.cuda.synchronize()
    st, info = c.solve_pressure(g, r, p, tol, max_iter=max_iter)
    torch.cuda.synchronize()
    return st, info, p.cpu().numpy()


# cells: one part full, one over; sheet and rod (few neighbours); one group
# full, one part over; three groups; uneven parts under random numbering
@pytest.mark.parametrize("shape,perm,kind,jitter", [
    ((16, 16, 16), None, "cavity", 0.0), ((17, 241, 1), 3, "cavity", 0.0), ((5000, 1, 1), None, "duct", 0.0),
    ((64, 64, 32), 5, "cavity", 0.0), ((65, 64, 32), None, "duct", 0.0), ((64, 72, 60), None, "cavity", 0.1)])
def test_against_oracle(shape, perm, kind, jitter):
    from paper_1207_1571_amd import fvm
    case = _case(shape, perm, kind, jitter)
    inputs = _inputs(case.mesh, 1)
    c = fvm.Case(case)
    oc = orc.OracleCase(case)
    for tol, max_iter in ((1e-3, 10000), (1e-12, 60)):
        st, info, p = _solve(c, inputs, tol, max_iter)
        po = inputs[2].copy()
        st_o, info_o = oc.solve_pressure(inputs[0], inputs[1], po, tol, max_iter=max_iter)
        err = np.linalg.norm(p - po) / np.linalg.norm(po)
        print(f"[resident] {shape} {kind} iters {info['iters']}/{info_o['iters']} rel {err:.1e}", file=sys.stderr, flush=True)
        assert st == st_o and info["iters"] == info_o["iters"]
        assert err <= TOL
        assert abs(info["res_final"] - info_o["res_final"]) <= 1e-6 * info_o["res_final"]


def test_solved_at_the_start_and_non_finite():
    """A guess that meets the tolerance takes no iteration and is returned
    as it is; a non-finite right-hand side fails without touching p."""
    from paper_1207_1571_amd import fvm
    case = _case((24, 20, 16), 2)
    gamma, rhs, p0 = _inputs(case.mesh, 2)
    c = fvm.Case(case)
    st, info, p = _solve(c, (gamma, rhs, p0), 10.0, 100)
    assert st == 0 and info["iters"] == 0 and np.array_equal(p, p0)
    bad = rhs.copy()
    bad[777] = np.nan
    with pytest.raises(fvm.FvmError) as e:
        _solve(c, (gamma, bad, p0), 1e-9, 100)
    assert e.value.code == fvm.FVM_ENUMERIC
    st, info, p = _solve(c, (gamma, rhs, p0), 1e-9, 1000)
    assert st == 0 and info["res_final"] <= 1e-9


def test_cases_sharing_launches_equal_their_own():
    """Cases of several sizes and stencils in one call (more parts than one
    launch holds): bit for bit what each computes alone."""
    from paper_1207_1571_amd import fvm
    specs = [_case((12, 10, 9), 1), _case((70, 70, 1), 2), _case((64, 64, 40)), _case((40, 30, 20), 3, "duct"),
             _case((90, 80, 70)), _case((96, 80, 70), None, "duct")]
    specs = [s.with_(step_kernel=wl.STEP_LAUNCHED, p_ctl=wl.SolverCtl(1e-5, max_iter=80), u_ctl=wl.SolverCtl(1e-6)) for s in specs]
    alone = []
    for s in specs:
        c = fvm.Case(s)
        c.piso(1)
        alone.append(c.get_state_numpy())
        c.close()
    cases = [fvm.Case(s) for s in specs]
    fvm.piso_batch(cases, 1)
    for c, a in zip(cases, alone):
        for x, y in zip(c.get_state_numpy(), a):
            assert np.array_equal(x, y)


def test_threads_and_streams():
    """Two threads solving on streams of their own at the same time."""
    import torch
    from paper_1207_1571_amd import fvm
    spec = _case((60, 50, 50))
    inputs = _inputs(spec.mesh, 4)
    ref = _solve(fvm.Case(spec), inputs, 1e-8, 500)[2]
    out, err = [None, None], []

    def work(k):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                c = fvm.Case(spec, stream=s)
                g, r, p0 = (torch.from_numpy(a.copy()).cuda() for a in inputs)
                for _ in range(5):
                    p = p0.clone()
                    c.solve_pressure(g, r, p, 1e-8, max_iter=500)
                out[k] = p.cpu().numpy()
        except Exception as e:   # noqa: BLE001
            err.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not err, err
    assert np.array_equal(out[0], ref) and np.array_equal(out[1], ref)


@pytest.mark.parametrize("static", [False, True])
def test_a_wait_that_runs_out(static):
    """A launch with a workgroup left out: the others' waits end, and the
    solve runs again from its start value as launched iterations."""
    import torch
    from paper_1207_1571_amd import fvm
    case = _case((64, 64, 40), 7)
    inputs = _inputs(case.mesh, 5)
    c = fvm.Case(case)
    hook = fvm.lib().fvm_resident_test_hook
    hook.argtypes = [ct.c_long, ct.c_int]
    hook.restype = None
    po = inputs[2].copy()
    _, info_o = orc.OracleCase(case).solve_pressure(inputs[0], inputs[1], po, 1e-12, max_iter=50)

    def once():
        g, r, p = (torch.from_numpy(a.copy()).cuda() for a in inputs)
        f = c.solve_pressure_static if static else c.solve_pressure
        st, info = f(g, r, p, 1e-12, max_iter=50)
        torch.cuda.synchronize()
        return st, info, p.cpu().numpy()

    hook(100000, 1)      # 1 ms
    try:
        st, info, p = once()
    finally:
        hook(0, 0)
    assert st == 1 and info["iters"] == info_o["iters"] == 50
    assert np.linalg.norm(p - po) / np.linalg.norm(po) <= TOL
    st, info, p = once()      # and the next solve is resident again
    assert st == 1 and info["iters"] == 50
    assert np.linalg.norm(p - po) / np.linalg.norm(po) <= TOL


def _hook():
    from paper_1207_1571_amd import fvm
    h = fvm.lib().fvm_resident_test_hook
    h.argtypes, h.restype = [ct.c_long, ct.c_int], None
    return h


# mixed precision, tile parts: one group; two; sheet; RCM numbering (columns
# explicit); a duct (fixed pressure); four groups
@pytest.mark.parametrize("shape,numbering,kind", [
    ((33, 33, 33), "lex", "cavity"), ((41, 47, 40), "lex", "duct"), ((230, 215, 1), "lex", "cavity"),
    ((40, 40, 40), "rcm", "cavity"), ((64, 64, 63), "lex", "cavity")])
def test_mixed_equals_the_launched_iterations(shape, numbering, kind):
    """The resident FP32 recurrence gives the launched iterations' bits (the
    launched side is reached by a launch whose wait runs out)."""
    from paper_1207_1571_amd import fvm
    case = _case(shape, None, kind).with_(precision=wl.MIXED)
    if numbering == "rcm":
        case = case.with_(mesh=mg.rcm(mg.random_permutation(case.mesh, 3)))
    inputs = _inputs(case.mesh, 6)
    c = fvm.Case(case)
    hook = _hook()
    for tol, max_iter in ((1e-6, 10000), (1e-9, 37)):
        hook(20000, 1)
        try:
            st_l, info_l, p_l = _solve(c, inputs, tol, max_iter)
        finally:
            hook(0, 0)
        st, info, p = _solve(c, inputs, tol, max_iter)
        print(f"[resident mixed] {shape} {numbering} iters {info['iters']}", file=sys.stderr, flush=True)
        assert st == st_l and info == info_l
        assert np.array_equal(p, p_l)


def test_mixed_cases_sharing_launches():
    from paper_1207_1571_amd import fvm
    specs = [_case((40, 40, 30)), _case((64, 64, 40), None, "duct"), _case((90, 80, 70)), _case((72, 72, 70), None, "duct"),
             _case((50, 40, 30), 4), _case((220, 200, 1))]
    specs = [s.with_(precision=wl.MIXED, p_ctl=wl.SolverCtl(1e-5, max_iter=60), u_ctl=wl.SolverCtl(1e-6)) for s in specs]
    alone = []
    for s in specs:
        c = fvm.Case(s)
        c.piso(1)
        alone.append(c.get_state_numpy())
        c.close()
    cases = [fvm.Case(s) for s in specs]
    fvm.piso_batch(cases, 1)
    for c, a in zip(cases, alone):
        for x, y in zip(c.get_state_numpy(), a):
            assert np.array_equal(x, y)


# DIC: one part; two; jagged parts of one group; three groups; sheet; cells
# with up to 6 lower neighbours (random numbering); a duct in its own order
@pytest.mark.parametrize("shape,numbering,kind", [
    ((16, 16, 16), "lex", "cavity"), ((17, 16, 16), "rcm", "cavity"), ((33, 31, 30), "rcm", "cavity"),
    ((66, 64, 63), "rcm", "cavity"), ((230, 90, 1), "random", "cavity"), ((40, 36, 30), "random", "cavity"),
    ((80, 30, 30), "lex", "duct")])
def test_dic_against_oracle(shape, numbering, kind):
    """And after a launch whose wait ran out, which leaves the solve to the
    launched sweeps.  25 iterations each: past some 100 iterations on a sheet
    the recurrence amplifies rounding (two runs of the launched sweeps then
    differ from each other by 3e-7)."""
    import torch
    from paper_1207_1571_amd import fvm
    case = _case(shape, None, kind).with_(p_ctl=wl.SolverCtl(1e-9, precond=wl.PC_DIC))
    if numbering != "lex":
        mesh = mg.random_permutation(case.mesh, 3)
        case = case.with_(mesh=mg.rcm(mesh) if numbering == "rcm" else mesh)
    inputs = _inputs(case.mesh, 7)
    c, oc, hook = fvm.Case(case), orc.OracleCase(case), _hook()
    for tol, max_iter, out in ((1e-12, 25, 0), (1e-12, 25, 1), (1e-12, 25, 0)):
        g, r, p = (torch.from_numpy(a.copy()).cuda() for a in inputs)
        torch.cuda.synchronize()
        if out and case.mesh.n_cells > 4096:   # of one part there is nothing to leave out
            hook(20000, 1)
        try:
            st, info = c.solve_pressure(g, r, p, tol, max_iter=max_iter, precond=wl.PC_DIC)
        finally:
            hook(0, 0)
        torch.cuda.synchronize()
        po = inputs[2].copy()
        st_o, info_o = oc.solve_pressure(inputs[0], inputs[1], po, tol, max_iter=max_iter, precond=wl.PC_DIC)
        err = np.linalg.norm(p.cpu().numpy() - po) / np.linalg.norm(po)
        print(f"[resident DIC] {shape} {numbering} iters {info['iters']}/{info_o['iters']} rel {err:.1e}", file=sys.stderr, flush=True)
        assert st == st_o and info["iters"] == info_o["iters"]
        assert err <= TOL


def test_dic_cases_sharing_launches():
    """Also with cases too large for the resident sweeps' parts next to them."""
    from paper_1207_1571_amd import fvm
    specs = [_case((12, 10, 9), 1), _case((70, 70, 1), 2), _case((64, 64, 40)), _case((90, 80, 70)),
             _case((96, 80, 70), None, "duct"), _case((104, 104, 104))]
    specs = [s.with_(step_kernel=wl.STEP_LAUNCHED, p_ctl=wl.SolverCtl(1e-5, max_iter=20, precond=wl.PC_DIC),
                     u_ctl=wl.SolverCtl(1e-6)) for s in specs]
    alone = []
    for s in specs:
        c = fvm.Case(s)
        c.piso(1)
        alone.append(c.get_state_numpy())
        c.close()
    cases = [fvm.Case(s) for s in specs]
    fvm.piso_batch(cases, 1)
    for k, (c, a) in enumerate(zip(cases, alone)):
        for x, y in zip(c.get_state_numpy(), a):
            assert np.linalg.norm(x - y) <= TOL * np.linalg.norm(y), k


def test_beside_whole_step_launches():
    """While whole-step launches hold CUs, resident solves are spread over the
    rest (or, in mixed precision, run as launched iterations): the same bits,
    a case of 256 parts included, which has to wait for them."""
    import torch
    from paper_1207_1571_amd import fvm
    small = [_case((12, 12, 12), k).with_(precision=wl.MIXED) for k in range(9)]
    specs = [_case((60, 50, 50)), _case((40, 40, 40)).with_(precision=wl.MIXED), _case((128, 96, 84)),
             _case((40, 36, 30), 3).with_(p_ctl=wl.SolverCtl(1e-9, precond=wl.PC_DIC))]
    inputs = [_inputs(s.mesh, 8) for s in specs]
    cases = [fvm.Case(s) for s in specs]

    def solve(k):
        g, r, p = (torch.from_numpy(a.copy()).cuda() for a in inputs[k])
        cases[k].solve_pressure(g, r, p, 1e-12, max_iter=30, precond=specs[k].p_ctl.precond)
        return p.cpu().numpy()

    ref = [solve(k) for k in range(len(specs))]
    stop, err, runs = threading.Event(), [], []

    def work():
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                cs = [fvm.Case(m, stream=s) for m in small]
                while not stop.is_set():
                    fvm.piso_batch(cs, 4)
                    runs.append(1)
        except Exception as e:   # noqa: BLE001
            err.append(e)

    t = threading.Thread(target=work)
    t.start()
    try:
        for _ in range(10):
            for k in range(len(specs)):
                assert np.array_equal(solve(k), ref[k]), k
    finally:
        stop.set()
        t.join()
    assert not err, err
    assert runs
