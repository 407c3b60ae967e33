"""Cells with more than 6 neighbours (hexagonal prisms): whole PISO steps in one
workgroup up to 4096 cells, launched phases above, against the oracle.

Tolerances: FP64 the parity bound 1e-9 (relative L2); mixed precision 1e-6
with an outer tolerance of 1e-10.
"""
import ctypes as ct
import sys

import numpy as np
import pytest

from oracle import oracle as orc
from paper_1207_1571_amd import workloads as wl
from tests import prisms

pytestmark = pytest.mark.gpu


def _steps(cases, n):
    """n steps of the cases in one call: fields, and whole-step launches made."""
    import torch
    from paper_1207_1571_amd import fvm
    cs = [fvm.Case(c) for c in cases]
    hook = fvm.lib().fvm_resident_test_hook   # a chip-filling solve of an earlier test is no longer about
    hook.argtypes, hook.restype = [ct.c_long, ct.c_int], None
    hook(0, 0)
    fvm.profile_enable(True)
    try:
        st, infos = fvm.piso_batch(cs, n)
        torch.cuda.synchronize()
    finally:
        fvm.profile_enable(False)
    assert st == 0
    out = [c.get_state_numpy() for c in cs]
    return out, infos, fvm.profile_read("solo_piso")[1]


# a remainder of a slice; several slices; the largest case of whole steps, and one over
@pytest.mark.parametrize("precision", [wl.FP64, wl.MIXED])
@pytest.mark.parametrize("shape,solo", [((9, 7, 5), 1), ((12, 11, 9), 1), ((16, 16, 16), 1), ((22, 17, 11), 0)])
def test_steps_against_oracle(shape, solo, precision):
    case = prisms.case(shape, precision, 1e-9 if precision == wl.FP64 else 1e-10)
    (g,), (info,), launches = _steps([case], 3)
    assert launches == solo
    (h,), _, launches = _steps([case.with_(step_kernel=wl.STEP_LAUNCHED)], 3)
    assert launches == 0
    oc = orc.OracleCase(case)
    st, info_o = oc.piso(3)
    assert st == 0
    tol = 1e-9 if precision == wl.FP64 else 1e-6
    for a, b, o in zip(g, h, (oc.U, oc.p, oc.phi)):
        e = [np.linalg.norm(x - o) / np.linalg.norm(o) for x in (a, b)]
        print(f"[prisms] {shape} precision {precision}: {e[0]:.1e} launched {e[1]:.1e}", file=sys.stderr, flush=True)
        assert max(e) <= tol
    if precision == wl.FP64:
        assert [k["iters"] for k in info["p"]] == [k["iters"] for k in info_o["p"]]


def test_both_kinds_of_cell_in_one_call():
    """Small mixed-precision cases of prisms and of hexahedra: a launch each,
    every case as it is alone."""
    specs = [prisms.case((9, 7, 5), wl.MIXED, 1e-6), wl.cavity((12, 11, 10), Re=100.0, dt=0.01, precision=wl.MIXED),
             prisms.case((6, 6, 6), wl.MIXED, 1e-6), wl.cavity((20, 20, 1), Re=100.0, dt=0.01, precision=wl.MIXED)]
    alone = [_steps([s], 2)[0][0] for s in specs]
    both, _, launches = _steps(specs, 2)
    assert launches == 2
    for a, b in zip(both, alone):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))
