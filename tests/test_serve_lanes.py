"""The lane of a served case follows the library's rule for whole steps."""
import threading

import pytest

from paper_1207_1571_amd import fvm, serve
from paper_1207_1571_amd import meshgen as mg
from paper_1207_1571_amd import workloads as wl
from tests import prisms


def _backend():
    """The backend's host side (its streams need a device)."""
    b = object.__new__(serve.GpuBackend)
    b.fvm, b._mu, b._meshes = fvm, threading.Lock(), {}
    return b


def _hexahedra(shape, **kw):
    return wl.cavity(shape, Re=100.0, dt=0.01).with_(**kw)


@pytest.mark.parametrize("spec,lane", [
    (_hexahedra((12, 11, 10), precision=wl.MIXED), "solo"), (_hexahedra((32, 32, 32), precision=wl.MIXED), "solo"),
    (_hexahedra((33, 32, 32), precision=wl.MIXED), "launched"), (_hexahedra((12, 11, 10)), "launched"),
    (prisms.case((9, 7, 5)), "solo"), (prisms.case((9, 7, 5), wl.MIXED), "solo"),
    (prisms.case((22, 17, 11), wl.MIXED), "launched"),
    (_hexahedra((12, 11, 10), precision=wl.MIXED, step_kernel=wl.STEP_LAUNCHED), "launched"),
    (_hexahedra((12, 11, 10), precision=wl.MIXED, mesh=mg.box_mesh(12, 11, 10, jitter=0.1, seed=1)), "launched"),
])
def test_lane(spec, lane):
    b = _backend()
    assert b.lane_of(spec) == lane          # of a case that was not priced
    b.footprint(spec)
    assert b.lane_of(spec) == lane


def test_lane_is_asked_while_the_priced_mesh_is_there():
    """create() takes the mesh that pricing made; the lane needs it too."""
    calls = []

    class Backend:
        LANES = {"solo": (4, 4), "launched": (4, 4)}

        def footprint(self, spec):
            calls.append("footprint")
            return 1

        def lane_of(self, spec):
            calls.append("lane_of")
            return "solo"

        def create(self, spec):
            calls.append("create")
            return spec

        def advance(self, cases, n, lane):
            return [dict(p=[], status=0) for _ in cases]

        def finish(self, case):
            return None

    res = serve.Server(Backend(), 10).run([serve.Request(0, 0.0, _hexahedra((4, 4, 4)), 2)])
    assert len(res) == 1 and calls == ["footprint", "lane_of", "create"]
