"""Autotuner of the FFT tile variants (points per thread, lines per
workgroup) of the row and column passes.

For every grid size present in a ``Propagator`` it times each compiled
variant of the forward row pass and of the forward column pass with the
library's HIP-event timing hook (``ssfm_time_passes``: launches on the
context's stream), keeps the fastest of each and selects them.  Results are
cached in a JSON file keyed by device name, grid size, precision and build of
the library (``SSFM_TUNE_CACHE``, default ``~/.cache/ssfm_tune.json``): a
variant is an index into that build's tiles, which another build may not have
or have for other tiles.
"""
from __future__ import annotations

import functools
import hashlib
import json
import os
from typing import Callable, Dict, List, Tuple

import torch

from . import _lib as L
from .march import Propagator, plan_variants


def _cache_path() -> str:
    return os.environ.get("SSFM_TUNE_CACHE",
                          os.path.join(os.path.expanduser("~"), ".cache", "ssfm_tune.json"))


@functools.lru_cache(maxsize=None)
def _build() -> str:
    with open(L.LIB_PATH, "rb") as f:
        return hashlib.sha256(f.read()).hexdigest()[:16]


def _key(n: int, precision: int) -> str:
    name = torch.cuda.get_device_name(0) if torch.cuda.is_available() else "none"
    return f"{name}|n={n}|fp{precision}|{_build()}"


def load_cache() -> Dict:
    try:
        with open(_cache_path()) as f:
            return json.load(f)
    except (OSError, ValueError):
        return {}


def save_cache(d: Dict) -> None:
    path = _cache_path()
    try:
        os.makedirs(os.path.dirname(path), exist_ok=True)
        with open(path, "w") as f:
            json.dump(d, f, indent=1)
    except OSError:
        pass


def _accepted(select: Callable[[int, int], None], row: int, col: int, refusals) -> bool:
    """Select a variant pair; False if the library refuses it."""
    try:
        select(row, col)
    except L.SsfmError as e:
        if e.status not in refusals:
            raise
        return False
    return True


def _times(select: Callable[[int, int], None], measure: Callable[[], Tuple[float, float]],
           n_row: int, n_col: int, base: int, refusals) -> Tuple[List, List]:
    """(time, variant) of every row and every column variant that the library
    accepts.  One measurement times a row and a column pass, which do not
    depend on each other: row variant v beside column variant v, or beside
    `base` where that pair is refused or there is no such column."""
    rows, cols = [], []
    for v in range(max(n_row, n_col)):
        if v < min(n_row, n_col) and _accepted(select, v, v, refusals):
            ms_row, ms_col = measure()
            rows.append((ms_row, v))
            cols.append((ms_col, v))
            continue
        if v < n_row and _accepted(select, v, base, refusals):
            rows.append((measure()[0], v))
        if v < n_col and _accepted(select, base, v, refusals):
            cols.append((measure()[1], v))
    return rows, cols


def _tune_adjoint(prop: Propagator, n: int, n_row: int, n_col: int, launches: int) -> Dict:
    """Adjoint-pass variants for size n among those with the forward
    variants' tiling (the library refuses the others)."""
    rows, cols = _times(lambda r, c: prop.select_adjoint_plan(n, r, c),
                        lambda: prop.time_adjoint_passes(launches)[::-1], n_row, n_col, -1,
                        (L.EINVAL, L.EUNSUPPORTED))
    br, bc = min(rows)[1], min(cols)[1]
    prop.select_adjoint_plan(n, br, bc)
    return {"row_adj": br, "col_adj": bc, "ms_row_adj": min(rows)[0], "ms_col_adj": min(cols)[0],
            "rows_adj_ms": {v: t for t, v in rows}, "cols_adj_ms": {v: t for t, v in cols}}


def tune(prop: Propagator, reps: int = 50, use_cache: bool = True,
         verbose: bool = False) -> Dict[int, Dict]:
    """Select the fastest row and column variants for each grid size of
    ``prop`` (and, for a context that can record, the fastest adjoint-pass
    variants with the same tiling) and return the timings.  reps: diffraction
    factors timed of each variant and axis; a launch holds two, so half as
    many launches.  The timing launches write the work buffer and the staging
    area only; the fields are unchanged."""
    launches = max(1, (reps + 1) // 2)
    cache = load_cache() if use_cache else {}
    out = {}
    for n in sorted({d.n for d in prop.descs}):
        key = _key(n, prop.precision)
        if use_cache and key in cache:
            best = cache[key]
            prop.select_plan(n, best["row"], best["col"])
            if prop.max_steps > 0 and "row_adj" in best:
                prop.select_adjoint_plan(n, best["row_adj"], best["col_adj"])
            out[n] = best
            continue
        n_row, n_col = plan_variants(n, prop.precision)
        # a variant whose tile does not fit a workgroup at this precision is
        # not built for it (EUNSUPPORTED) and is skipped
        rows, cols = _times(lambda r, c: prop.select_plan(n, r, c),
                            lambda: prop.time_passes(launches)[:2], n_row, n_col, 0,
                            (L.EUNSUPPORTED,))
        br, bc = min(rows)[1], min(cols)[1]
        prop.select_plan(n, br, bc)
        best = {"row": br, "col": bc, "ms_row": min(rows)[0], "ms_col": min(cols)[0],
                "rows_ms": [r[0] for r in rows], "cols_ms": [c[0] for c in cols]}
        if prop.max_steps > 0:
            best.update(_tune_adjoint(prop, n, n_row, n_col, launches))
        if verbose:
            print(f"tune n={n} fp{prop.precision}: rows(us)="
                  f"{[round(r[0] * 1e3, 2) for r in rows]} cols(us)="
                  f"{[round(c[0] * 1e3, 2) for c in cols]} -> row {br}, col {bc}", flush=True)
        cache[key] = best
        out[n] = best
    if use_cache:
        save_cache(cache)
    return out
