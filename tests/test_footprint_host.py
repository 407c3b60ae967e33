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
