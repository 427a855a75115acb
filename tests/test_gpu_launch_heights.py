"""The strip height of the 2D stage a caller sets, or the autotuner times and
reports, is the one that runs; 0 is the library's own choice.  Heights are
told apart by the stage's time: on a small grid a launch lasts as long as one
strip's row steps."""
import numpy as np
import pytest

from paper_2201_12193_amd import autotune
from paper_2201_12193_amd import inputs as I

pytestmark = pytest.mark.gpu


def _solver(nx=96, ny=96):
    import torch
    from paper_2201_12193_amd.mrhweno import Solver
    print(f"heights: {nx}x{ny}", flush=True)
    rng = np.random.default_rng(2)
    prob = I.Problem(dim=2, nx=nx, ny=ny, x1=nx / ny, t_final=float("inf"))
    U = np.zeros(prob.shape())
    r, p = rng.uniform(0.95, 1.05, (2, ny, nx))
    U[:, 0] = I.euler2d_cons(r, 0.3 * r, 0.1 * p, p, 1.4)
    return Solver([prob], [torch.from_numpy(U).cuda()])


def _stage_ms(s):
    """Mean time of a stage launch (least of five)."""
    out = []
    for _ in range(5):
        ms, nl = s.profile(2)
        out.append(ms[3] / nl[3])
    return min(out)


def test_set_height_runs():
    """96 x 96: a strip of all 96 rows takes 98 row steps one after another,
    one of 8 rows 10."""
    s = _solver()
    s.profile(1)
    own = _stage_ms(s)
    t = {}
    for rows in (8, 32, 96):
        s.set_launch(rows, 0)
        t[rows] = _stage_ms(s)
    print(f"heights: own {own} {t}", flush=True)
    assert t[96] > 2.0 * t[32] > 4.0 * t[8] and t[8] > 1.5 * own
    s.set_launch(0, 0)
    again = _stage_ms(s)
    s.close()
    assert abs(again - own) < 0.3 * own


def test_autotune_reports_what_runs():
    s = _solver()
    rows, grid, ms = s.autotune(rows=(96, 8, 32), grids=(0,), reps=10)
    assert (rows, grid) == (8, 0)
    assert abs(_stage_ms(s) - ms) < 0.5 * ms
    s.close()


@pytest.mark.parametrize("rows", [-1, 1, 7, 4097])
def test_heights_out_of_range_are_refused(rows):
    from paper_2201_12193_amd.mrhweno import ERR_INVALID_ARG, MrError
    s = _solver(16, 16)
    with pytest.raises(MrError) as e:
        s.set_launch(rows, 0)
    assert e.value.status == ERR_INVALID_ARG
    s.close()


@pytest.mark.parametrize("nx,ny", [(96, 96), (512, 512), (331, 257)])
def test_tune_does_not_lose_to_the_own_choice(nx, ny, tmp_path, monkeypatch):
    monkeypatch.setattr(autotune, "CACHE", str(tmp_path / "autotune.json"))
    s = _solver(nx, ny)
    s.profile(1)
    default = _stage_ms(s)
    s.set_launch(96, 0)
    first = autotune.tune(s)
    tuned = _stage_ms(s)
    s.set_launch(96, 0)
    hit = autotune.tune(s)
    assert hit.ms is None and hit[:2] == first[:2] and hit.kx_rows == first.kx_rows
    cached = _stage_ms(s)
    s.close()
    print(f"heights: default {default} tuned {tuned} cached {cached} {first}", flush=True)
    assert tuned < 1.25 * default and cached < 1.25 * default
    # what tune returns can be set on another solver
    s = _solver(nx, ny)
    s.set_launch(*first[:2])
    s.close()
