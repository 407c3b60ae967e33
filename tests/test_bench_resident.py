"""The benchmark's figures where pressure solves run resident: time per
iteration, and assembly against a product measured by itself."""
import os
import sys

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


class _Fvm:
    """Kernel classes of two steps of a resident DIC case: 4 solves, 100
    iterations in all, 36 ms."""
    TIMES = {"pcg_dic_resident": (36.0, 4), "mom_face": (0.1, 2), "mom_cell": (0.2, 2), "bicg_spmv": (1.0, 30)}

    def profile_enable(self, on):
        pass

    def profile_read(self, cls):
        return self.TIMES.get(cls, (0.0, 0))


class _Case:
    def piso(self, n):
        return 0, dict(p=[dict(iters=30), dict(iters=20)], u=[dict(iters=7), dict(iters=9), dict(iters=8)])


@pytest.fixture(autouse=True)
def no_device(monkeypatch):
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)


def test_resident_solves_are_counted_in_iterations():
    k = bench.profile_classes(_Fvm(), _Case(), 2, 1000, 2700, True, None)
    r = k["pcg_dic_resident"]
    assert r["launches"] == 4 and r["work_launches"] == 100
    assert abs(r["us_per_work"] - 360.0) < 1e-9 and abs(r["mean_us"] - 9000.0) < 1e-9
    assert k["bicg_spmv"]["work_launches"] == 18
    assert bench.dic_figures(k) == {"pcg_dic_resident": dict(us_per_work=360.0, alg_GBps=None, counter_bytes=None)}


def test_assembly_against_the_product_alone():
    k = bench.profile_classes(_Fvm(), _Case(), 2, 1000, 2700, True, None)
    k["op_spmv"] = dict(us_per_work=25.0)
    a = bench.vs_spmv(k, "op_spmv")
    assert a["momentum assembly (convection + Laplacian: mom_face + mom_cell)"] == 6.0   # (50 + 100) / 25
    assert a["flux correction (flux_corr)"] is None
