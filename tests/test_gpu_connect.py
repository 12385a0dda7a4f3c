"""Connectivity of the pore space on the GPU against SciPy's labelling (needs an MI355X).

Random voxels near the percolation threshold (long, branching, mostly disconnected paths) on
boxes around the kernels' 64-cell row segments and 256-cell blocks, and a winding channel whose
single path visits every other row.  The count of unconnected cells is a whole number: equal.
"""
import re

import numpy as np
import pytest
import torch
from scipy import ndimage

pytestmark = pytest.mark.gpu


def unconnected(sv, solid):
    """The count the library reports (0 if it accepts the geometry)."""
    try:
        sv.setup_geometry(torch.as_tensor(solid, device="cuda"))
        return 0
    except sv.SocfvError as e:
        assert e.code == sv.BAD_GEOMETRY
        return int(re.search(r"(\d+) pore cells", str(e)).group(1))


def expected(solid):
    lab, _ = ndimage.label(solid == 0)
    inlet = np.unique(lab[:, :, 0])
    return int(((lab > 0) & ~np.isin(lab, inlet[inlet > 0])).sum())


@pytest.fixture(scope="module")
def sv():
    from paper_2502_08034_amd import socfv
    assert torch.cuda.is_available()
    return socfv


@pytest.mark.parametrize("nx,ny,nz", [(2, 1, 1), (63, 5, 4), (64, 5, 4), (65, 5, 4), (129, 17, 9),
                                      (200, 30, 31), (7, 300, 11), (256, 64, 80)])
@pytest.mark.parametrize("fill", [0.3, 0.65, 0.69, 0.8])
def test_random_voxels(sv, nx, ny, nz, fill):
    rng = np.random.Generator(np.random.PCG64(nx + 1000 * ny + int(100 * fill)))
    solid = (rng.random((nz, ny, nx)) < fill).astype(np.uint8)
    solid[0, 0, 0] = solid[-1, -1, -1] = 0          # a pore cell at the inlet and the outlet
    assert unconnected(sv, solid) == expected(solid)


@pytest.mark.parametrize("cut", [False, True])
def test_winding_channel(sv, cut):
    # rows y = 0, 2, 4, ... open from end to end, joined at alternating ends: one path
    solid = np.ones((3, 41, 150), dtype=np.uint8)
    solid[1, ::2, 1:] = 0
    for k, y in enumerate(range(1, 41, 2)):
        solid[1, y, -1 if k % 2 == 0 else 1] = 0
    solid[1, 0, 0] = 0
    if cut:
        solid[1, 20, 75] = 1
    want = expected(solid)
    assert (want > 0) == cut
    assert unconnected(sv, solid) == want


def test_the_labels_take_no_memory_of_their_own(sv):
    # a context holds 1 B a cell of flags, and with a velocity 36 B of faces; the 4 B a cell of the
    # labels are the x faces' (or given back by the flow step), so no sum has them on top
    nx, ny, nz = 256, 256, 192
    n, slack = nx * ny * nz, 16 << 20
    solid = torch.zeros((nz, ny, nx), dtype=torch.uint8, device="cuda")
    u = [torch.zeros(s, dtype=torch.float64, device="cuda")
         for s in ((nz, ny, nx + 1), (nz, ny + 1, nx), (nz + 1, ny, nx))]
    u[0].fill_(1.0)
    torch.cuda.synchronize()

    def held(ctx_of):
        before = torch.cuda.mem_get_info()[0]
        ctx = ctx_of()
        torch.cuda.synchronize()
        used = before - torch.cuda.mem_get_info()[0]
        del ctx
        return used

    def with_velocity():
        ctx = sv.setup_geometry(solid)
        sv.set_velocity(ctx, *u)
        return ctx

    def after_flow():
        ctx = sv.setup_geometry(solid)
        sv.solve_stokes(ctx, start=[*u, None], max_steps=1, cg_max=1, tol=0.0)
        return ctx

    assert held(with_velocity) <= 37 * n + slack
    assert held(after_flow) <= n + slack
