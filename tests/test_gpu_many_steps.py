"""Steps replayed several at a time give what single steps give, bit for bit:
counts around the eight steps of one replay, and a final time that falls
inside a replay."""
import numpy as np
import pytest

from paper_2201_12193_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsteps", [1, 7, 8, 9, 17])
@pytest.mark.parametrize("clip", [False, True])
@pytest.mark.parametrize("n", [24, 64])
def test_same_as_single_steps(n, clip, nsteps):
    import torch
    from paper_2201_12193_amd.mrhweno import Solver
    prob, U, _ = I.euler_quadrants_2d(seed=13, n=n, nq=2)
    print(f"many steps: n={n} clip={clip} steps={nsteps}", flush=True)
    Ut = torch.from_numpy(np.ascontiguousarray(U)).cuda()
    if clip:   # after about half the steps
        s = Solver([prob.replace(t_final=float("inf"))], [Ut.clone()])
        s.step((nsteps + 1) // 2)
        t, _, _ = s.sync()
        s.close()
        prob = prob.replace(t_final=0.98 * t[0])
    else:
        prob = prob.replace(t_final=float("inf"))
    out = []
    for single in (False, True):
        Us = Ut.clone()
        s = Solver([prob], [Us])
        for k in [1] * nsteps if single else [nsteps]:
            s.step(k)
        t, steps, st = s.sync()
        s.close()
        out.append((t[0], steps[0], Us.cpu().numpy()))
    assert out[0][:2] == out[1][:2]
    assert np.array_equal(out[0][2], out[1][2])
