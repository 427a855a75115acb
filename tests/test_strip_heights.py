"""Work-list sizes of the 2D stage strips: the height the library chooses by
itself (and the lower strips along a side with boundary data) stays within
the workspace mrhweno_workspace_bytes asks for.  Runs where a GPU is; the
states come back equal whatever the height."""
import numpy as np
import pytest

from paper_2201_12193_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(8, 8), (63, 9), (96, 96), (200, 7 * 62), (331, 257), (1024, 40)])
def test_heights_agree(nx, ny):
    import torch
    from paper_2201_12193_amd.mrhweno import Solver
    print(f"heights: {nx}x{ny}", flush=True)
    rng = np.random.default_rng(1)
    prob = I.Problem(dim=2, nx=nx, ny=ny, x1=nx / ny, bc_x=I.TRANSMISSIVE, bc_y=I.PERIODIC)
    U = np.zeros(prob.shape())
    r, p = rng.uniform(0.9, 1.1, (2, ny, nx))
    U[:, 0] = I.euler2d_cons(r, 0.3 * r, 0.1 * p, p, 1.4)
    out = []
    for rows in (0, 8, 11, 4096):
        Ut = torch.from_numpy(U).cuda()
        s = Solver([prob], [Ut])
        if rows:
            s.set_launch(rows, 0)
        s.step(2)
        s.sync()
        s.close()
        out.append(Ut.cpu().numpy())
    for o in out[1:]:
        assert np.array_equal(out[0], o)


def test_lower_strips_along_sides_fit():
    """Inflow on the left: the strips along it take half the rows."""
    import torch
    from paper_2201_12193_amd.mrhweno import Solver
    prob, U = I.double_mach_2d(ny=24)
    out = []
    for rows in (0, 8, 40):
        Ut = torch.from_numpy(U).cuda()
        s = Solver([prob], [Ut])
        if rows:
            s.set_launch(rows, 0)
        s.step(2)
        s.sync()
        s.close()
        out.append(Ut.cpu().numpy())
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
