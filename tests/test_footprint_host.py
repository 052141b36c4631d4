"""The device memory of a handle, counted on the host: programs set a server's
budget to what their meshes take, so a handle takes no more than it did."""
import pytest

import paper_0912_1976_amd as lib
from inputs import box_mesh


# bytes taken while the preconditioner's two cycles still had fine sweeps of their own
@pytest.mark.parametrize("nx,ny,nz,mode,pc,taken", [
    (25, 25, 17, "D", "vl_as", 16305656), (29, 27, 9, "N", "vl_sor", 15189796), (33, 31, 2, "N", "vl_as", 6700240),
    (41, 37, 5, "R", "vl_as", 18975164), (21, 19, 9, "N", "sa", 9601616)])
def test_a_handle_takes_no_more_memory_than_before(nx, ny, nz, mode, pc, taken):
    m = box_mesh(nx, ny, nz, 1e-2, jitter=0.3, seed=nx, bathymetry=True)
    s = lib.Solver(m.xyz, m.tets, m.top, top_bc=mode, device=-1, pc=pc, coarse_max=256,
                   robin_alpha=20.0 if mode == "R" else 0.0)
    assert s.footprint() <= taken
