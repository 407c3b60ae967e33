"""Which kernels a pressure solve runs: the resident ones where a case has
parts for them, launched iterations after a wait that ran out, and then for a
while without trying again.
"""
import ctypes as ct

import numpy as np
import pytest

from paper_1207_1571_amd import workloads as wl

pytestmark = pytest.mark.gpu
RESIDENT = ("pcg_resident", "pcg32_resident", "pcg_dic_resident")
LAUNCHED = ("pcg_spmv", "pcg32_spmv")
LEAVE_OUT, REMEMBER = 1, 2


@pytest.fixture
def hook():
    from paper_1207_1571_amd import fvm
    h = fvm.lib().fvm_resident_test_hook
    h.argtypes, h.restype = [ct.c_long, ct.c_int], None
    yield h
    h(0, 0)


def _ran(f):
    """The classes of CG kernels that f launches."""
    import torch
    from paper_1207_1571_amd import fvm
    fvm.profile_enable(True)
    try:
        f()
        torch.cuda.synchronize()
    finally:
        fvm.profile_enable(False)
    return {k for k in RESIDENT + LAUNCHED if fvm.profile_read(k)[1] > 0}


class _Pressure:
    def __init__(self, shape, precision=wl.FP64, precond=wl.PC_JACOBI, static=False):
        import torch
        from paper_1207_1571_amd import fvm
        spec = wl.cavity(shape, Re=100.0, dt=0.01, precision=precision, p_precond=precond)
        rng = np.random.default_rng(3)
        rhs = rng.normal(size=spec.mesh.n_cells)
        self.p0 = rng.normal(size=spec.mesh.n_cells)
        self.g, self.r, self.p = (torch.from_numpy(a).cuda() for a in
                                  (rng.uniform(0.5, 2.0, spec.mesh.n_faces), rhs - rhs.mean(), self.p0.copy()))
        self.case, self.precond, self.static = fvm.Case(spec), precond, static

    def __call__(self):
        import torch
        self.p.copy_(torch.from_numpy(self.p0))
        torch.cuda.synchronize()
        if self.static:
            self.case.solve_pressure_static(self.g, self.r, self.p, 1e-8, max_iter=20)
        else:
            self.case.solve_pressure(self.g, self.r, self.p, 1e-8, max_iter=20, precond=self.precond)
        return self.p.cpu().numpy()


KINDS = [(wl.FP64, wl.PC_JACOBI, False, "pcg_resident", "pcg_spmv"), (wl.FP64, wl.PC_JACOBI, True, "pcg_resident", "pcg_spmv"),
         (wl.FP64, wl.PC_DIC, False, "pcg_dic_resident", "pcg_spmv"), (wl.MIXED, wl.PC_JACOBI, False, "pcg32_resident", "pcg32_spmv")]


@pytest.mark.parametrize("precision,precond,static,resident,launched", KINDS)
def test_the_resident_kernel_runs(hook, precision, precond, static, resident, launched):
    s = _Pressure((40, 40, 40), precision, precond, static)
    assert _ran(s) == {resident}
    hook(20000, LEAVE_OUT)
    assert _ran(s) == {resident, launched}
    hook(0, 0)
    assert _ran(s) == {resident}


@pytest.mark.parametrize("precision,precond,static,resident,launched", KINDS)
def test_a_wait_that_ran_out_is_remembered(hook, precision, precond, static, resident, launched):
    s = _Pressure((40, 40, 40), precision, precond, static)
    one = _Pressure((12, 12, 12))     # of one part: waits for no other workgroup
    ref = s()
    hook(20000, LEAVE_OUT | REMEMBER)
    assert _ran(s) == {resident, launched}
    late = s()
    hook(10 ** 9, REMEMBER)           # the usual limit, nothing left out
    assert _ran(s) == {launched}
    # the launched DIC sweeps sum r.z by the blocks that claimed the tiles: their bits differ from run to run
    if precond == wl.PC_DIC:
        assert np.linalg.norm(s() - late) <= 1e-9 * np.linalg.norm(late)
    else:
        assert np.array_equal(s(), late)
    assert _ran(one) == {"pcg_resident"}
    hook(0, 0)                        # forgotten
    assert _ran(s) == {resident}
    assert np.array_equal(s(), ref)


def test_a_batch_while_it_is_remembered(hook):
    """Cases of one part solve resident, the others of the call launched; and
    all resident again later, in the same order of sums."""
    from paper_1207_1571_amd import fvm
    specs = [wl.cavity(n, Re=100.0, dt=0.01, tol=1e-5) for n in ((12, 12, 12), (40, 40, 40), (10, 9, 8), (30, 30, 30))]

    def step(n=1):
        cases = [fvm.Case(s) for s in specs]
        out = []
        ran = _ran(lambda: out.append(fvm.piso_batch(cases, n)))
        return ran, [c.get_state_numpy() for c in cases]

    ran, ref = step()
    assert ran == {"pcg_resident"}
    big = _Pressure((40, 40, 40))
    hook(20000, LEAVE_OUT | REMEMBER)
    big()
    hook(10 ** 9, REMEMBER)
    ran, mixed = step()
    assert ran == {"pcg_resident", "pcg_spmv"}
    for k in (0, 2):
        assert all(np.array_equal(a, b) for a, b in zip(mixed[k], ref[k])), k
    for k in (1, 3):
        assert all(np.linalg.norm(a - b) <= 1e-9 * np.linalg.norm(b) for a, b in zip(mixed[k], ref[k])), k
    hook(0, 0)
    ran, again = step()
    assert ran == {"pcg_resident"}
    assert all(np.array_equal(a, b) for x, y in zip(again, ref) for a, b in zip(x, y))


@pytest.mark.parametrize("precision,precond", [(wl.FP64, wl.PC_JACOBI), (wl.FP64, wl.PC_DIC), (wl.MIXED, wl.PC_JACOBI)])
def test_a_failed_solve_leaves_p(precision, precond):
    import torch
    from paper_1207_1571_amd import fvm
    s = _Pressure((40, 40, 40), precision, precond)
    s.r[777] = float("nan")
    with pytest.raises(fvm.FvmError) as e:
        s()
    assert e.value.code == fvm.FVM_ENUMERIC
    torch.cuda.synchronize()
    assert np.array_equal(s.p.cpu().numpy(), s.p0)
