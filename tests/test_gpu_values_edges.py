"""The one-off reconstruction where waves of interior cells, which load their
stencils at fixed offsets, and waves with cells at an edge, which load them
by the ghost rules, meet: grids whose rows are a few waves long, every
boundary condition, values and flags against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2201_12193_amd import inputs as I
from tests.parity_util import TOL, comp_scale

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["burgers", "euler", "char"])
@pytest.mark.parametrize("tc", [I.TC_ALL, I.TC_KXRCF, I.TC_NONE])
@pytest.mark.parametrize("bc", [I.PERIODIC, I.TRANSMISSIVE, I.REFLECTIVE])
def test_values(bc, tc, kind):
    import torch
    from paper_2201_12193_amd.mrhweno import Solver
    if kind == "burgers" and bc == I.REFLECTIVE:
        pytest.skip("walls: Euler only")
    print(f"values: {kind} bc={bc} tc={tc}", flush=True)
    nx, ny = 256, 9
    rng = np.random.default_rng(4)
    prob = I.Problem(dim=2, nx=nx, ny=ny, x1=nx / ny, bc_x=bc, bc_y=bc, tc_mode=tc,
                     system=I.BURGERS if kind == "burgers" else I.EULER, charwise=1 if kind == "char" else 0)
    U = np.zeros(prob.shape())
    r, p = rng.uniform(0.6, 1.4, (2, ny, nx))
    u, v = rng.uniform(-0.4, 0.4, (2, ny, nx))
    if kind == "burgers":
        U[0, 0] = u
    else:
        U[:, 0] = I.euler2d_cons(r, u, v, p, 1.4)
    U[:, 1:] = 0.02 * rng.uniform(-1, 1, U[:, 1:].shape)
    Ut = torch.from_numpy(U).cuda()
    s = Solver([prob], [Ut.clone()])
    gl, fl = s.reconstruct(0, Ut)
    s.close()
    ref, flref, _, _ = oracle.reconstruct(prob, U)
    d = np.abs(gl.cpu().numpy() - ref).reshape(prob.ncomp, -1).max(axis=1) / comp_scale(prob, U)
    assert d.max() <= TOL, d
    assert np.array_equal(fl.cpu().numpy(), flref)
