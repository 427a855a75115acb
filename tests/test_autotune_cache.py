"""The autotuner's cache: shapes are kept per kind of problem and build of the
library, and an entry of another kind, or of a file written before the kind
was part of the key, is timed again."""
import json
from types import SimpleNamespace

import pytest

from paper_2201_12193_amd import autotune, mrhweno
from paper_2201_12193_amd import inputs as I


class Fake:
    """A solver's launch-shape calls, recorded."""

    def __init__(self, *problems):
        self.problems = problems
        self.timed = 0
        self.applied = None

    def autotune(self, rows, grids, reps):
        self.timed += 1
        return 16, 0, 0.5

    def autotune_indicator(self, rows, reps):
        return 8, 0.1

    def set_launch(self, rows, grid):
        self.applied = (rows, grid)

    def set_indicator_launch(self, rows):
        self.applied += (rows,)


@pytest.fixture
def cache(tmp_path, monkeypatch):
    lib = tmp_path / "lib.so"
    lib.write_bytes(b"one build")
    monkeypatch.setattr(mrhweno, "LIB_PATH", str(lib))
    monkeypatch.setattr(autotune, "CACHE", str(tmp_path / "autotune.json"))
    monkeypatch.setattr(autotune, "_arch", lambda: "gfx950")
    yield SimpleNamespace(lib=lib, file=tmp_path / "autotune.json")


BASE = I.Problem(dim=2, nx=64, ny=64)
OTHERS = [BASE.replace(charwise=1), BASE.replace(beta_on=I.BETA_ON_P), BASE.replace(tc_mode=I.TC_NONE),
          I.Problem(dim=2, nx=64, ny=64, system=I.BURGERS), I.double_mach_2d(ny=32)[0], BASE.replace(nx=128, ny=128)]   # (the last: another size)


def test_same_kind_is_not_timed_again(cache):
    a, b = Fake(BASE), Fake(BASE.replace(nx=65, ny=65, x1=1.0))
    autotune.tune(a, grids=(0,))
    assert a.timed == 1
    assert autotune.tune(b, grids=(0,)) == (16, 0, None, 8)
    assert b.timed == 0 and b.applied == (16, 0, 8)


@pytest.mark.parametrize("k", range(len(OTHERS)))
def test_other_kind_is_timed(cache, k):
    autotune.tune(Fake(BASE), grids=(0,))
    o = Fake(OTHERS[k])
    autotune.tune(o, grids=(0,))
    assert o.timed == 1


def test_mixed_batch_is_timed(cache):
    autotune.tune(Fake(BASE), grids=(0,))
    autotune.tune(Fake(OTHERS[0]), grids=(0,))
    o = Fake(BASE, OTHERS[0])
    autotune.tune(o, grids=(0,))
    assert o.timed == 1


def test_other_build_is_timed(cache, monkeypatch):
    autotune.tune(Fake(BASE), grids=(0,))
    other = cache.lib.with_name("other.so")
    other.write_bytes(b"another build")
    monkeypatch.setattr(mrhweno, "LIB_PATH", str(other))
    o = Fake(BASE)
    autotune.tune(o, grids=(0,))
    assert o.timed == 1


def test_entries_of_an_older_file_are_not_applied(cache):
    cache.file.write_text(json.dumps({"gfx950/dim2/nc4/cells2^12": {"rows": 32, "grid": 0, "kx_rows": 46}}))
    s = Fake(BASE)
    assert autotune.tune(s, grids=(0,)).rows == 16
    assert s.timed == 1 and s.applied is None
