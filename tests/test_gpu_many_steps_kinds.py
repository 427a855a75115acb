"""Steps replayed several at a time, for the kinds of instances whose steps
hand something from launch to launch besides the state: the learned
indicator's list of undecided cells, the alpha of 1D Burgers stages, and
batches of all of them with 1D and 2D instances of both systems."""
import numpy as np
import pytest

from paper_2201_12193_amd import inputs as I

pytestmark = pytest.mark.gpu


def _learned(n=96, **kw):
    prob, U, _ = I.euler_quadrants_2d(seed=13, n=n, nq=2)
    return prob.replace(tc_mode=I.TC_LEARNED, t_final=float("inf"), **kw), U


def _plain(n=48):
    prob, U, _ = I.euler_quadrants_2d(seed=14, n=n, nq=2)
    return prob.replace(t_final=float("inf")), U


def _burgers1(n=200, **kw):
    prob, U, _ = I.burgers_smooth_1d(seed=7, n=n)
    return prob.replace(t_final=float("inf"), **kw), U


def _euler1(n=300, **kw):
    prob, U, _ = I.euler_riemann_1d(3, n=n)
    return prob.replace(t_final=float("inf"), **kw), U


def _burgers2(n=40):
    prob = I.Problem(dim=2, nx=n, ny=n, system=I.BURGERS, t_final=float("inf"))
    x = (np.arange(n) + 0.5) / n
    U = np.zeros(prob.shape())
    U[0, 0] = 0.2 + np.sin(2 * np.pi * (x[None, :] + x[:, None]))
    return prob, U


KINDS = {
    "learned": lambda: [_learned()],
    "learned_p": lambda: [_learned(beta_on=I.BETA_ON_P)],
    "burgers1": lambda: [_burgers1()],
    "burgers1_tiles": lambda: [_burgers1(777, tc_mode=I.TC_ALL)],
    "burgers12": lambda: [_burgers1(), _burgers2(), _burgers1(501)],
    "mixed": lambda: [_learned(), _burgers1(), _euler1(), _plain(), _burgers2(), _euler1(500, charwise=1)],
}


@pytest.mark.parametrize("nsteps", [8, 9, 17])
@pytest.mark.parametrize("kind", KINDS)
def test_same_as_single_steps(kind, nsteps):
    """Three passes on the same solver (eager set-up work between them), each
    equal to single steps bit for bit."""
    import torch
    from paper_2201_12193_amd.indicator import DEFAULT_BAND, load_weights
    from paper_2201_12193_amd.mrhweno import Solver
    print(f"many steps: {kind} {nsteps}", flush=True)
    cases = KINDS[kind]()
    starts = [torch.from_numpy(np.ascontiguousarray(U)).cuda() for _, U in cases]
    out = []
    for single in (True, False):
        Us = [U.clone() for U in starts]
        s = Solver([p for p, _ in cases], Us)
        if any(p.tc_mode == I.TC_LEARNED for p, _ in cases):
            s.set_indicator(load_weights(), *DEFAULT_BAND)
        for _ in range(3):
            for q, (a, b) in enumerate(zip(Us, starts)):
                a.copy_(b)
                s.set_time(q, 0.0, 0)
            torch.cuda.synchronize()
            for k in [1] * nsteps if single else [nsteps]:
                s.step(k)
            t, n, st = s.sync()
            assert st == 0
            out.append((list(t), list(n), [a.cpu().numpy() for a in Us]))
        s.close()
    for o in out[1:]:
        assert o[0] == out[0][0] and o[1] == out[0][1]
        assert all(np.array_equal(a, b) for a, b in zip(o[2], out[0][2]))
