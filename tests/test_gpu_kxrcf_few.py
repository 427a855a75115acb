"""The one-wave KXRCF kernel of small launches: columns at the edges of its
strips (62 flag columns of the range [-2, n+2)), the boundary conditions,
both smoothness-indicator variants and Step 1 variants, other linear
weights, and states whose velocities take every branch: of one sign
throughout (no Step 1 of the momenta), at rest, and of mixed signs by rows
and by columns (a row without a sign next to one with it reconstructs the
lower row late).  Flags equal to the oracle's bit for bit (the bar of the
other parity tests); steps equal bit for bit with those of k2_kxrcf, which a
height set by the caller selects (the flags are all that differs between
the two)."""
import numpy as np
import pytest

import oracle
from paper_2201_12193_amd import inputs as I

pytestmark = pytest.mark.gpu


def _problem(nx, ny, vel, bc, beta_on, char):
    rng = np.random.default_rng(nx + 7 * ny)
    prob, _, _ = I.euler_quadrants_2d(seed=5, n=64, nq=2)
    prob = prob.replace(nx=nx, ny=ny, x1=prob.x0 + prob.dx * nx, y1=prob.y0 + prob.dy * ny, bc_x=bc, bc_y=bc,
                        beta_on=I.BETA_ON_P if beta_on else I.BETA_ON_Q, charwise=char)
    if beta_on:
        prob = prob.replace(gbar=(1.0, 2.5, 7.0, 40.0), eps=1e-6)
    return prob, rng


def _state(prob, rng, vel):
    ny, nx = prob.ny, prob.nx
    y, x = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
    rho = 1.0 + 0.3 * np.sin(0.4 * x + 0.2 * y) + 0.5 * (x > nx // 2) + 0.4 * (y > ny // 2)
    one = np.ones_like(rho)
    u, v = {"moving": (one, -one), "rest": (0 * one, 0 * one), "rows": (np.where(y % 3 == 0, 1.0, -1.0), np.where(y % 4 < 2, 0.8, -0.8)),
            "columns": (np.where(x % 5 < 2, 1.0, -1.0), np.where(x == nx // 3, -1.0, 1.0)),
            "noise": tuple(rng.standard_normal((2, ny, nx)))}[vel]
    U = np.zeros((4, 3, ny, nx))
    U[0, 0], U[1, 0], U[2, 0] = rho, rho * u, rho * v
    U[3, 0] = 1.5 / 0.4 + 0.5 * rho * (u * u + v * v)
    U[:, 1:] = 0.02 * rng.standard_normal((4, 2, ny, nx))
    return U


CASES = [(8, 8, "noise", I.PERIODIC, 0, 0), (58, 9, "rows", I.TRANSMISSIVE, 0, 0), (59, 70, "columns", I.REFLECTIVE, 0, 0),
         (62, 33, "moving", I.PERIODIC, 1, 0), (63, 40, "rest", I.REFLECTIVE, 0, 0), (120, 31, "rows", I.PERIODIC, 1, 0),
         (121, 300, "columns", I.TRANSMISSIVE, 0, 0), (200, 200, "noise", I.PERIODIC, 0, 0), (244, 200, "rows", I.PERIODIC, 0, 0),
         (331, 257, "columns", I.PERIODIC, 1, 0), (430, 400, "rows", I.TRANSMISSIVE, 0, 0),
         (59, 33, "rows", I.REFLECTIVE, 0, 1), (121, 64, "noise", I.PERIODIC, 1, 1)]


@pytest.mark.parametrize("nx,ny,vel,bc,beta_on,char", CASES)
def test_flags(nx, ny, vel, bc, beta_on, char):
    import torch
    from paper_2201_12193_amd.mrhweno import Solver
    print(f"kxrcf few: {nx} x {ny} {vel} bc={bc} beta={beta_on} char={char}", flush=True)
    prob, rng = _problem(nx, ny, vel, bc, beta_on, char)
    U = _state(prob, rng, vel)
    _, fref = oracle.residual(prob, U)
    Ut = torch.from_numpy(U).cuda()
    s = Solver([prob], [Ut.clone()])
    fl, _ = s.flag(0, Ut)
    s.close()
    assert np.array_equal(fl.cpu().numpy(), fref)
    out = []
    for rows in (0, 8):
        Us = Ut.clone()
        s = Solver([prob], [Us])
        s.set_indicator_launch(rows)
        s.step(2)
        s.sync(raise_on_error=False)
        s.close()
        out.append(Us.cpu().numpy())
    assert np.array_equal(out[0], out[1], equal_nan=True)
