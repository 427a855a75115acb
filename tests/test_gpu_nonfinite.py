"""States with NaN, infinite or zero entries: the one-off residual leaves
finite what the formulas leave finite (the oracle's pattern), with the same
flags, and the finite values agree to the bar of the other parity tests."""
import numpy as np
import pytest

import oracle
from paper_2201_12193_amd import inputs as I
from tests.parity_util import TOL, comp_scale

pytestmark = pytest.mark.gpu


def _base(prob, seed=7):
    """Random averages around a moderate state, small random first moments."""
    rng = np.random.default_rng(seed)
    shp = prob.shape()[2:]
    U = np.zeros(prob.shape())
    r, p = rng.uniform(0.8, 1.2, (2,) + shp)
    u, v = rng.uniform(-0.3, 0.3, (2,) + shp)
    U[:, 0] = I.euler1d_cons(r, u, p, 1.4) if prob.dim == 1 else I.euler2d_cons(r, u, v, p, 1.4)
    U[:, 1:] = 0.01 * rng.uniform(-1, 1, U[:, 1:].shape)
    return U


def _run(tag, prob, U, clean):
    """GPU and oracle residual and flags, and the scale of the residual."""
    import torch
    from paper_2201_12193_amd.mrhweno import Solver
    print(f"nonfinite: {tag}", flush=True)
    Ut = torch.from_numpy(np.ascontiguousarray(U)).cuda()
    s = Solver([prob], [Ut.clone()])
    R, fl = s.residual(0, Ut)
    s.close()
    with np.errstate(all="ignore"):
        Lref, flref = oracle.residual(prob, U)
    scale = comp_scale(prob, clean) / oracle.dt(prob, clean)
    return R.cpu().numpy(), fl.cpu().numpy(), Lref, flref, scale.reshape((-1,) + (1,) * (U.ndim - 1))


def _check(R, Lref, scale):
    fin = np.isfinite(Lref)
    assert np.array_equal(np.isfinite(R), fin)
    assert (np.abs(R - Lref)[fin] <= TOL * (scale + np.abs(Lref))[fin]).all()


@pytest.mark.parametrize("bc", [I.PERIODIC, I.REFLECTIVE])
@pytest.mark.parametrize("value", [np.nan, np.inf, 0.0])
def test_mass_flux_where_the_density_is_undefined_1d(value, bc):
    """The mass flux of a state whose density is NaN, infinite or zero is its
    momentum: the density's residual stays finite."""
    prob = I.Problem(dim=1, nx=30, bc_x=bc, tc_mode=I.TC_NONE)
    clean = _base(prob)
    U = clean.copy()
    if value == 0.0:
        U[0, :, 12:15] = 0.0   # zero at every point of the middle cell
    else:
        U[0, 0, 12] = value
    R, fl, Lref, flref, scale = _run(f"mass flux 1d density={value} bc={bc}", prob, U, clean)
    assert np.isfinite(Lref[0]).all() and not np.isfinite(Lref[1:]).all()
    _check(R[:1], Lref[:1], scale[:1])


@pytest.mark.parametrize("case", ["kxrcf", "none", "all", "tvb", "beta_p", "reflective", "transmissive"])
@pytest.mark.parametrize("comp,value", [(3, np.nan), (3, np.inf), (3, -np.finfo(float).max), (2, np.nan), (1, np.nan)])
def test_component_of_a_cell_2d(comp, value, case):
    """One average that is not finite: the components, cells and faces that do
    not depend on it keep their values (the volume and face sums of the 2D
    stage kernel run over all components of a cell together)."""
    kw = {"none": dict(tc_mode=I.TC_NONE), "all": dict(tc_mode=I.TC_ALL), "tvb": dict(tc_mode=I.TC_TVB),
          "beta_p": dict(beta_on=I.BETA_ON_P), "reflective": dict(bc_x=I.REFLECTIVE, bc_y=I.REFLECTIVE),
          "transmissive": dict(bc_x=I.TRANSMISSIVE, bc_y=I.TRANSMISSIVE)}.get(case, {})
    prob = I.Problem(dim=2, nx=24, ny=20, x1=1.2, **kw)
    clean = _base(prob)
    for at in ((0, 0), (9, 10)):
        U = clean.copy()
        U[(comp, 0) + at] = value
        R, fl, Lref, flref, scale = _run(f"2d {case} component {comp} = {value} at {at}", prob, U, clean)
        assert not np.isfinite(Lref).all() and np.isfinite(Lref[0]).any()
        _check(R, Lref, scale)
        assert np.array_equal(fl, flref)


@pytest.mark.parametrize("nx", [130, 700])
def test_alpha_beside_a_block_of_nan_1d(nx):
    """1D Burgers with NaN first moments over more than a wave's cells: the
    Lax-Friedrichs alpha of stages 2 and 3 comes from the other cells, which
    the step advances as the oracle does."""
    import torch
    from paper_2201_12193_amd.mrhweno import Solver
    print(f"nonfinite: alpha nx={nx}", flush=True)
    prob = I.Problem(dim=1, nx=nx, system=I.BURGERS, tc_mode=I.TC_NONE)
    U = np.zeros(prob.shape())
    U[0, 0] = 0.3 + np.sin(2 * np.pi * (np.arange(nx) + 0.5) / nx)
    clean = U.copy()
    U[0, 1, 40:128] = np.nan
    Ut = torch.from_numpy(U.copy()).cuda()
    s = Solver([prob], [Ut])
    s.step(1)
    dt = s.last_dt()[0]
    s.sync(raise_on_error=False)
    s.close()
    with np.errstate(all="ignore"):
        ref = oracle.rk3_step(prob, U, dt)
    fin = np.isfinite(ref)
    assert fin[0, 0, 5:30].all() and not fin[0, 0, 50:120].any()
    got = Ut.cpu().numpy()
    assert np.array_equal(np.isfinite(got), fin)
    assert np.abs(got - ref)[fin].max() <= TOL * comp_scale(prob, clean)[0]


@pytest.mark.parametrize("nx", [24, 70])
@pytest.mark.parametrize("bc", [I.PERIODIC, I.REFLECTIVE, I.TRANSMISSIVE])
@pytest.mark.parametrize("comp,value", [(0, np.nan), (0, np.inf), (0, 0.0), (0, -0.1), (1, np.inf), (2, np.nan),
                                        (2, -np.inf), (1, 1e200), (0, 1e-300)])
def test_flags_beside_a_state_that_is_not_physical_2d(comp, value, bc, nx):
    """The KXRCF strips of small grids leave out the momenta's Step 1 where
    bounds decide the velocities' signs: a value that is not finite, or no
    positive density, takes the full path, and the flags are the oracle's."""
    prob = I.Problem(dim=2, nx=nx, ny=20, x1=nx / 20, bc_x=bc, bc_y=bc)
    clean = _base(prob)
    clean[1, 0] += 0.9 * clean[0, 0]   # mostly one sign: the bounds decide
    clean[2, 0] -= 0.9 * clean[0, 0]
    clean[3, 0] += 1.0
    for at in ((0, 0), (9, 10)):
        U = clean.copy()
        U[(comp, 0) + at] = value
        R, fl, Lref, flref, scale = _run(f"flags component {comp} = {value} at {at} bc={bc} nx={nx}", prob, U, clean)
        assert np.array_equal(fl, flref)
