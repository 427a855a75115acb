"""The learned indicator's strips at the edges of their tiles (64 columns,
steps of four rows, one to several strips high) with every cell left to the
KXRCF test, so that the list of undecided cells overflows its place in LDS:
all decisions are 2, and the flags are those of the KXRCF indicator except
where its two sides agree to rounding (both kernels sum a few hundred terms:
1e-12 of either side)."""
import pytest

import numpy as np

from paper_2201_12193_amd import inputs as I
from tests.test_gpu_learned import _learned_solver, _params, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,bc", [(8, 8, I.PERIODIC), (60, 61, I.TRANSMISSIVE), (61, 9, I.REFLECTIVE),
                                      (125, 130, I.PERIODIC), (200, 333, I.REFLECTIVE), (700, 640, I.TRANSMISSIVE)])
def test_every_cell_undecided(nx, ny, bc):
    from paper_2201_12193_amd.mrhweno import Solver
    print(f"learned strips: {nx} x {ny} bc={bc}", flush=True)
    n = max(nx, ny)
    prob, U, _ = I.euler_quadrants_2d(seed=11, n=n + n % 2, nq=2)
    U = np.ascontiguousarray(U[:, :, :ny, :nx])
    prob = prob.replace(nx=nx, ny=ny, x1=prob.x0 + prob.dx * nx, y1=prob.y0 + prob.dy * ny, bc_x=bc, bc_y=bc)
    s = Solver([prob], [_t(U)])
    fk, al = s.flag(0, _t(U))
    s.close()
    s, Ut, _ = _learned_solver(prob, U, _params(3), 0.0, 1.0)
    dec, fl = s.indicator(0, Ut)
    s.close()
    assert (dec.cpu().numpy() == 2).all()
    num, den = al[..., 0].cpu().numpy(), al[..., 1].cpu().numpy()
    close = np.abs(num - den) <= 1e-12 * (num + den)
    assert ((fl.cpu().numpy() == fk.cpu().numpy()) | close).all()
