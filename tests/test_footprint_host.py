"""What a case's workspace holds: parts of the resident solves for cases that
solve with them, not for AMG cases."""
import pytest

from paper_1207_1571_amd import fvm
from paper_1207_1571_amd import meshgen as mg
from paper_1207_1571_amd import workloads as wl


@pytest.mark.parametrize("precond,same", [(wl.PC_JACOBI, False), (wl.PC_AMG, True)])
def test_amg_cases_hold_no_parts(precond, same):
    """The parts follow the cells' places: stretching the box cuts it otherwise,
    with other halos.  Nothing else in a workspace depends on the geometry."""
    sizes = []
    for z in (1.0, 100.0):
        case = wl.cavity((32, 24, 20), Re=100.0, dt=0.01, p_precond=precond)
        case = case.with_(mesh=mg.box_mesh(32, 24, 20, lengths=(1.0, 1.0, z)))
        sizes.append(fvm.workspace_bytes(fvm.Mesh(case.mesh, case.bcs), fvm.opts_from_case(case)))
    assert (sizes[0] == sizes[1]) == same, sizes


def test_range_of_the_static_solve(tmp_path):
    """solve_pressure_static takes cases of up to 10 995 712 cells and refuses
    larger ones (its scratch is 4 MiB)."""
    import os
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    (tmp_path / "main.cpp").write_text(r'''
#include <cstdio>
#include "fvm_internal.h"
int main()
{
    for (long N : {1L, 8000000L, 10995712L, 10995713L, 11008000L}) {
        const int32_t s = (int32_t)(((N + kBlock - 1) / kBlock + 7) / 8 * 8);   // the plan's strides
        std::printf("%d ", (int)(static_counted_bytes(s, (s + kGroup - 1) / kGroup) <= kStaticScratchBytes));
    }
}
''')
    exe = str(tmp_path / "range")
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                           os.path.join(root, "include"), "-I", os.path.join(root, "paper_1207_1571_amd", "csrc"),
                           str(tmp_path / "main.cpp"), "-o", exe])
    assert subprocess.check_output([exe], text=True).split() == ["1", "1", "1", "0", "0"]
