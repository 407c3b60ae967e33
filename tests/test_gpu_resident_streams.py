"""Resident pressure solves on several streams: launches share the device where
the CUs suffice, wait for each other where they do not, and give the bits that
each gives alone.
"""
import ctypes as ct
import sys
import threading

import numpy as np
import pytest

from paper_1207_1571_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _case(shape):
    return wl.duct(shape, mode="piso", dt=0.01) if shape[1] == 1 else wl.cavity(shape, Re=100.0, dt=0.01)


def _inputs(mesh, seed):
    rng = np.random.default_rng(seed)
    rhs = rng.normal(size=mesh.n_cells)
    return rng.uniform(0.5, 2.0, mesh.n_faces), rhs - rhs.mean(), rng.normal(size=mesh.n_cells) * 0.1


class _Solver:
    """A case on a stream of its own."""

    def __init__(self, shape, seed):
        import torch
        from paper_1207_1571_amd import fvm
        self.stream = torch.cuda.Stream()
        with torch.cuda.stream(self.stream):
            spec = _case(shape)
            self.case = fvm.Case(spec, stream=self.stream)
            self.g, self.r, self.p0 = (torch.from_numpy(a).cuda() for a in _inputs(spec.mesh, seed))
        self.stream.synchronize()

    def solve(self, max_iter):
        """max_iter iterations (the tolerance is out of reach)"""
        import torch
        with torch.cuda.stream(self.stream):
            p = self.p0.clone()
            st, info = self.case.solve_pressure(self.g, self.r, p, 0.0, max_iter=max_iter)
            assert st == 1 and info["iters"] == max_iter
            return p.cpu().numpy()


# one part (a workgroup that waits for nobody); one group of 4 parts
@pytest.mark.parametrize("cells", [4096, 16384])
def test_small_solves_run_side_by_side(cells):
    """While one stream runs solves of 4000 iterations (a rod, which takes as
    many to converge), another ends many of 20 in the time of each.  (Two
    streams may share one of the 4 hardware queues, where everything runs in
    order: four further streams are tried.)"""
    long = _Solver((cells, 1, 1), 1)
    long_ref = long.solve(4000)
    runs, counts = 20, []
    for _ in range(5):
        short = _Solver((cells, 1, 1), 2)
        ref, err, started = short.solve(20), [], threading.Event()

        def work():
            try:
                for _ in range(runs):
                    started.set()
                    assert np.array_equal(long.solve(4000), long_ref)
            except BaseException as e:   # noqa: BLE001
                err.append(e)

        t = threading.Thread(target=work)
        t.start()
        started.wait()
        n = 0
        while t.is_alive():
            assert np.array_equal(short.solve(20), ref)
            n += 1
        t.join()
        assert not err, err
        counts.append(n)
        if n >= 3 * runs:
            break
    print(f"[streams] {cells} cells: {counts} short solves beside {runs} long ones", file=sys.stderr, flush=True)
    assert counts[-1] >= 3 * runs, counts


def test_solves_of_all_sizes_on_many_streams():
    """More CUs asked for than there are: one to 256 parts on six streams."""
    shapes = [(128, 96, 84), (16, 16, 16), (64, 64, 40), (24, 24, 24), (60, 50, 50), (12, 12, 12)]
    solvers = [_Solver(s, k) for k, s in enumerate(shapes)]
    ref = [s.solve(40) for s in solvers]
    err = []

    def work(k):
        try:
            for _ in range(12):
                assert np.array_equal(solvers[k].solve(40), ref[k]), k
        except BaseException as e:   # noqa: BLE001
            err.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(len(solvers))]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not err, err


@pytest.fixture
def forgetful():
    """What the library remembers of crowded launches ends with the test."""
    from paper_1207_1571_amd import fvm
    yield
    h = fvm.lib().fvm_resident_test_hook
    h.argtypes, h.restype = [ct.c_long, ct.c_int], None
    h(0, 0)


def test_large_solves_find_their_turn_beside_whole_steps(forgetful):
    """A case that needs nearly all CUs solves between the steps of whole-step
    calls, not once per call; both give the bits they give alone.  One of the
    small cases fails in its first step: it stays as it is, the others go on."""
    import torch
    from paper_1207_1571_amd import fvm
    big = _Solver((128, 96, 84), 5)           # 252 parts
    ref = big.solve(20)
    spec = wl.cavity((24, 24, 24), Re=100.0, dt=0.005, precision=wl.MIXED)
    mesh = fvm.Mesh(spec.mesh, spec.bcs)
    calls, steps, bad, stream = 3, 40, 5, torch.cuda.Stream()

    def cases():
        with torch.cuda.stream(stream):
            cs = [fvm.Case(spec.with_(nu=0.01 + 0.001 * k), stream=stream, mesh=mesh) for k in range(32)]
            cs[bad].set_state(U=torch.full((cs[bad].n_cells, 3), float("nan"), dtype=torch.float64, device="cuda"))
        stream.synchronize()
        return cs

    def run(cs):
        with torch.cuda.stream(stream):
            return [fvm.piso_batch(cs, steps, stream=stream, raise_on_case_failure=False)[1] for _ in range(calls)]

    one, two = cases(), cases()
    infos = run(one)
    out, err, n = [], [], 0

    def work():
        try:
            out.append(run(two))
        except BaseException as e:   # noqa: BLE001
            err.append(e)

    t = threading.Thread(target=work)
    t.start()
    while t.is_alive():
        assert np.array_equal(big.solve(20), ref)
        n += 1
    t.join()
    print(f"[streams] {n} large solves beside {calls} calls of {steps} whole steps", file=sys.stderr, flush=True)
    assert not err, err
    for a, b in zip(out[0], infos):
        assert a[bad]["status"] == b[bad]["status"] == fvm.FVM_ENUMERIC
        assert a[:bad] + a[bad + 1:] == b[:bad] + b[bad + 1:]
    for a, b in zip(one, two):
        assert all(np.array_equal(x, y, equal_nan=True) for x, y in zip(a.get_state_numpy(), b.get_state_numpy()))
    # one or two per call without that; where the two streams share a hardware
    # queue, a solve's own round trips each pass a step: some 7 per call
    assert n >= 4 * calls, n
