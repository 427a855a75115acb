"""The 2D stage kernel at the edges of its strips (a strip owns 62 Euler or
254 Burgers columns and stages two more each side) and the branches of its
HLLC flux, against the oracle: residual within 1e-12 of each component's
scale over dt, flags bit for bit (the bars of the other parity tests)."""
import numpy as np
import pytest

import oracle
from paper_2201_12193_amd import inputs as I
from tests.parity_util import comp_scale

pytestmark = pytest.mark.gpu
TOL = 1e-12


def _residual(prob, U):
    import torch
    from paper_2201_12193_amd.mrhweno import Solver
    print(f"stage2d: {prob.nx}x{prob.ny} system={prob.system} bc={prob.bc_x} tc={prob.tc_mode}", flush=True)
    Ut = torch.from_numpy(np.ascontiguousarray(U)).cuda()
    s = Solver([prob], [Ut.clone()])
    R, fl = s.residual(0, Ut)
    s.close()
    Lref, flref = oracle.residual(prob, U)
    d = np.abs(R.cpu().numpy() - Lref).reshape(prob.ncomp, -1).max(axis=1) / (comp_scale(prob, U) / oracle.dt(prob, U))
    assert d.max() <= TOL, d
    assert np.array_equal(fl.cpu().numpy(), flref)
    return flref


def _euler(nx, ny, bc, seed=3):
    """Random smooth-free Euler data (jumps everywhere): every cell's branch differs."""
    rng = np.random.default_rng(seed)
    prob = I.Problem(dim=2, nx=nx, ny=ny, x1=nx / ny, bc_x=bc, bc_y=bc)
    r, p = rng.uniform(0.5, 1.5, (2, ny, nx))
    u, v = rng.uniform(-0.5, 0.5, (2, ny, nx))
    U = np.zeros(prob.shape())
    U[:, 0] = I.euler2d_cons(r, u, v, p, 1.4)
    U[:, 1:] = 0.02 * rng.uniform(-1, 1, (4, 2, ny, nx))
    return prob, U


@pytest.mark.parametrize("bc", [I.PERIODIC, I.TRANSMISSIVE, I.REFLECTIVE])
@pytest.mark.parametrize("nx", [8, 61, 62, 63, 66, 124, 125])
def test_strip_edges(nx, bc):
    prob, U = _euler(nx, 9, bc)
    assert _residual(prob, U).any()


@pytest.mark.parametrize("nx", [253, 254, 255, 258, 509])
def test_strip_edges_burgers(nx):
    rng = np.random.default_rng(5)
    prob = I.Problem(dim=2, nx=nx, ny=10, x1=nx / 10.0, system=I.BURGERS)
    U = np.zeros(prob.shape())
    U[0, 0] = rng.uniform(-1.0, 1.0, (10, nx))
    U[0, 1:] = 0.05 * rng.uniform(-1, 1, (2, 10, nx))
    assert _residual(prob, U)[:, 240:].any()


@pytest.mark.parametrize("axis", [0, 1])
def test_hllc_left_speed_positive_with_a_leftgoing_contact(axis):
    """Colliding streams whose estimated contact speed is negative while the
    left wave speed is not: the flux is the left state's."""
    n = 16
    prob = I.Problem(dim=2, nx=n, ny=n, bc_x=I.TRANSMISSIVE, bc_y=I.TRANSMISSIVE, tc_mode=I.TC_NONE)
    left = np.arange(n) < n // 2
    p = 1.0 / 1.4
    r, vn, pr = np.ones(n), np.where(left, 2.5, -2.45), np.where(left, p, p + 0.2)
    line = I.euler2d_cons(r, vn, 0.3 * r, pr, 1.4)
    if axis == 1:
        line = line[[0, 2, 1, 3]]
    U = np.zeros(prob.shape())
    U[:, 0] = line[:, None, :] if axis == 0 else line[:, :, None]
    fL = oracle.hllc(line[:, n // 2 - 1], line[:, n // 2], 1.4, axis)
    q = line[:, n // 2 - 1]
    phys = q * 2.5
    phys[1 + axis] += p
    phys[3] += 2.5 * p
    assert np.allclose(fL, phys, rtol=1e-14)      # the branch 0 <= sL
    rc = 0.5 * (1.0 + np.sqrt(1.4 * (p + 0.2)))   # mean density 1 times the mean sound speed
    assert 0.05 - 0.2 / rc < 0.0                  # s* < 0
    _residual(prob, U)
