"""Launch-shape autotuning with a persistent cache.

The C ABI's mrhweno_autotune times candidate 2D launch shapes of the stage
kernel on the instances' current states (without advancing them) and applies
the fastest; mrhweno_autotune_indicator does the same for the strip height of
the 2D KXRCF pass.  This module remembers the choices per GPU architecture,
build of the library, kernel variants of the problems and problem-size bucket
in a JSON file, so later contexts of the same kind apply them without
re-timing."""
from __future__ import annotations

import functools
import hashlib
import json
import math
import os
from typing import NamedTuple, Optional

from . import inputs
from . import mrhweno

CACHE = os.path.join(os.path.expanduser(os.environ.get("MRHWENO_CACHE_DIR", "~/.cache/mrhweno")),
                     "autotune.json")
ROWS = (0, 8, 16, 24, 32, 40, 48, 56, 64, 72, 96)
KX_ROWS = (0, 8, 16, 24, 32, 46, 64, 96, 140)   # 0 in both: the height the library chooses by size


class Launch(NamedTuple):
    rows: int          # rows per work item of the 2D stage kernel (0: by size)
    grid: int          # its grid (0: one work group per work item)
    ms: Optional[float]
    kx_rows: int       # flag rows per work item of the 2D KXRCF pass (0: by size)


def _arch() -> str:
    import torch
    p = torch.cuda.get_device_properties(0)
    return getattr(p, "gcnArchName", p.name).split(":")[0]


@functools.lru_cache(maxsize=None)
def _build(path: str) -> str:
    """Hash of the built library: shapes timed with other kernels do not apply."""
    with open(path, "rb") as f:
        return hashlib.sha1(f.read()).hexdigest()[:12]


def _variant(p) -> str:
    """The kernels an instance takes: components, Step 1, smoothness
    indicators, troubled-cell mode, data on the sides or a step."""
    data = "d" if p.step_j > 0 or inputs.SIDES in (p.bc_x, p.bc_y) else ""
    return f"nc{p.ncomp}{'c' if p.charwise else ''}{'p' if p.beta_on == inputs.BETA_ON_P else ''}t{p.tc_mode}{data}"


def key(solver) -> str:
    """arch / build / dim / variants of the 2D instances / log2 bucket of
    their total cell count"""
    two = [p for p in solver.problems if p.dim == 2]
    cells = sum(p.ncell for p in two)
    bucket = int(math.log2(max(cells, 1)))
    variants = "+".join(sorted({_variant(p) for p in two}))
    return f"{_arch()}/{_build(mrhweno.LIB_PATH)}/dim2/{variants}/cells2^{bucket}"


def _load() -> dict:
    try:
        with open(CACHE) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def resident_grid() -> int:
    """Work groups of the 2D stage kernel that fit the GPU at once (two per
    compute unit)."""
    import torch
    return 2 * torch.cuda.get_device_properties(0).multi_processor_count


def tune(solver, use_cache: bool = True, grids=None, reps: int = 3) -> Launch:
    """Apply the cached launch shapes for this kind of problem, or time the
    candidates (stage kernel: strip heights ROWS and grids, one work group
    per work item and a persistent grid of resident size unless given;
    KXRCF pass: strip heights KX_ROWS), apply the fastest and cache them.
    ms is the stage kernel's mean launch time (None for a cache hit)."""
    if grids is None:
        grids = (0, resident_grid())
    k = key(solver)
    db = _load()
    if use_cache and k in db and "kx_rows" in db[k]:
        e = db[k]
        solver.set_launch(e["rows"], e["grid"])
        solver.set_indicator_launch(e["kx_rows"])
        return Launch(e["rows"], e["grid"], None, e["kx_rows"])
    rows, grid, ms = solver.autotune(rows=ROWS, grids=grids, reps=reps)
    kx_rows, kx_ms = solver.autotune_indicator(rows=KX_ROWS, reps=reps)
    db[k] = {"rows": rows, "grid": grid, "ms": ms, "kx_rows": kx_rows, "kx_ms": kx_ms}
    try:
        os.makedirs(os.path.dirname(CACHE), exist_ok=True)
        tmp = CACHE + ".tmp"
        with open(tmp, "w") as f:
            json.dump(db, f, indent=1, sort_keys=True)
        os.replace(tmp, CACHE)
    except OSError:
        pass
    return Launch(rows, grid, ms, kx_rows)
