"""Host memory that runs out while a case is planned: an error code, no C++
exception past the interface (it would end the process), and the same call
succeeds once there is memory again.

The address space of a child process is limited after the mesh is made; large
blocks come from mmap there, so that nothing freed earlier serves them.
"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes as ct, resource, sys
sys.path.insert(0, %r)
from paper_1207_1571_amd import fvm, workloads as wl
precond, precision = int(sys.argv[1]), int(sys.argv[2])
case = wl.cavity((60, 60, 60), Re=100.0, dt=0.01, precision=precision, p_precond=precond)
mesh, opts, L = fvm.Mesh(case.mesh, case.bcs), fvm.opts_from_case(case), fvm.lib()
n, h = ct.c_size_t(), ct.c_void_p()
ws = ct.create_string_buffer(4096)
at = (ct.addressof(ws) + 255) // 256 * 256
size = lambda: L.fvm_case_workspace_bytes(mesh.handle, ct.byref(opts), ct.byref(n))
create = lambda: L.fvm_case_create(mesh.handle, ct.byref(opts), at, 1, None, ct.byref(h))
vm = 4096 * int(open('/proc/self/statm').read().split()[0])
resource.setrlimit(resource.RLIMIT_AS, (vm + (1 << 20), resource.RLIM_INFINITY))
a = size(), L.fvm_last_error(), create(), L.fvm_last_error(), h.value
resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY, resource.RLIM_INFINITY))
b = size(), create(), h.value
print(a, b, n.value > 60 ** 3 * 500, flush=True)
assert a == (-2, b'out of memory', -2, b'out of memory', None), a
assert b == (0, -2, None), b          # the buffer given is one byte
assert b'too small' in L.fvm_last_error()
"""


# FP64 Jacobi and DIC, AMG, mixed precision
@pytest.mark.parametrize("precond,precision", [(0, 0), (1, 0), (2, 0), (0, 1)])
def test_planning_without_memory(precond, precision):
    env = dict(os.environ, MALLOC_MMAP_THRESHOLD_="65536", MALLOC_ARENA_MAX="1", OMP_NUM_THREADS="1")
    r = subprocess.run([sys.executable, "-c", CHILD % ROOT, str(precond), str(precision)], capture_output=True, text=True,
                       timeout=300, env=env)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-2000:])
