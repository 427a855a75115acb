"""Steps of the 2D stage kernel against the oracle over the whole grid at set
strip heights: strips of several rows (the LDS rings wrap, the top trace is
carried from row to row), a short last strip, one strip over all rows, and
the library's own height (one or two rows here).  Grids two strips wide and
43 rows high; every height gives the same bits."""
import numpy as np
import pytest

import oracle
from paper_2201_12193_amd import inputs as I
from tests.parity_util import TOL, comp_scale, rel_state_err

pytestmark = pytest.mark.gpu
HEIGHTS = ((0, 0), (8, 0), (13, 0), (32, 3), (64, 0))   # rows, grid


def _euler(nx=70, ny=43, seed=5, **kw):
    rng = np.random.default_rng(seed)
    prob = I.Problem(dim=2, nx=nx, ny=ny, x1=nx / ny, t_final=float("inf"), **kw)
    U = np.zeros(prob.shape())
    r, p = rng.uniform(0.7, 1.3, (2, ny, nx))
    u, v = rng.uniform(-0.4, 0.4, (2, ny, nx))
    U[:, 0] = I.euler2d_cons(r, u, v, p, 1.4)
    U[:, 1:] = 0.02 * rng.uniform(-1, 1, (4, 2, ny, nx))
    return prob, U


def _burgers(nx=300, ny=43, **kw):
    rng = np.random.default_rng(6)
    prob = I.Problem(dim=2, nx=nx, ny=ny, x1=nx / ny, system=I.BURGERS, t_final=float("inf"), **kw)
    U = np.zeros(prob.shape())
    U[0, 0] = rng.uniform(-1, 1, (ny, nx))
    U[0, 1:] = 0.05 * rng.uniform(-1, 1, (2, ny, nx))
    return prob, U


def _later(prob, U, steps=8, **kw):
    """A problem with data on its sides after some of the oracle's steps, its
    time set back to 0 (the fronts start anew: a state like any other)."""
    prob = prob.replace(t_final=float("inf"), **kw)
    for _ in range(steps):
        U = oracle.rk3_step(prob, U, oracle.dt(prob, U))
    return prob, U


P, T, R = I.PERIODIC, I.TRANSMISSIVE, I.REFLECTIVE
CASES = {
    "euler": lambda: _euler(),
    "euler_transmissive": lambda: _euler(bc_x=T, bc_y=T),
    "euler_walls": lambda: _euler(bc_x=R, bc_y=R),
    "euler_mixed": lambda: _euler(bc_x=T, bc_y=P, modification=I.MOD_INTERNAL),
    "euler_stage_mod": lambda: _euler(modification=I.MOD_STAGE),
    "euler_all": lambda: _euler(tc_mode=I.TC_ALL),
    "euler_none": lambda: _euler(tc_mode=I.TC_NONE),
    "euler_tvb": lambda: _euler(tc_mode=I.TC_TVB),
    "euler_p": lambda: _euler(beta_on=I.BETA_ON_P, bc_y=R),
    "char": lambda: _euler(charwise=1),
    "char_walls": lambda: _euler(charwise=1, bc_x=R, bc_y=T),
    "char_p": lambda: _euler(charwise=1, beta_on=I.BETA_ON_P, tc_mode=I.TC_ALL),
    "burgers": lambda: _burgers(),
    "burgers_transmissive": lambda: _burgers(bc_x=T, bc_y=T),
    "burgers_p": lambda: _burgers(beta_on=I.BETA_ON_P, tc_mode=I.TC_ALL),
    "dmr": lambda: _later(*I.double_mach_2d(ny=43)),
    "dmr_p": lambda: _later(*I.double_mach_2d(ny=43), beta_on=I.BETA_ON_P),
    "fstep": lambda: _later(*I.forward_step(ny=45)),
    "fstep_char": lambda: _later(*I.forward_step(ny=45), charwise=1),
}


@pytest.mark.parametrize("name", CASES)
def test_steps(name):
    import torch
    from paper_2201_12193_amd.mrhweno import Solver
    prob, U = CASES[name]()
    sc = comp_scale(prob, U)
    dt = oracle.dt(prob, U)
    ref = oracle.rk3_step(prob, U, dt)
    out = []
    for rows, grid in HEIGHTS:
        print(f"step heights: {name} {prob.nx}x{prob.ny} rows={rows} grid={grid}", flush=True)
        Ut = torch.from_numpy(np.ascontiguousarray(U)).cuda()
        s = Solver([prob], [Ut])
        if rows:
            s.set_launch(rows, grid)
        s.step(1)
        assert s.last_dt()[0] == dt
        s.sync()
        one = Ut.cpu().numpy()
        assert rel_state_err(prob, one, ref, sc) <= TOL
        s.step(1)
        s.sync()
        s.close()
        out.append(np.stack([one, Ut.cpu().numpy()]))
        assert np.array_equal(out[0], out[-1]), rows
