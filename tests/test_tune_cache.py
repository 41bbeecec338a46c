"""The tuner on a stand-in for a context: what it measures, and its cache file,
whose entries belong to one library file."""
import json

import pytest

from paper_2306_15678_amd import _lib as L
from paper_2306_15678_amd import tune as tuner
from paper_2306_15678_amd.march import make_desc

N = 1024


class _Context:
    """A context as the tuner sees it: two variants of each pass, the second
    one the faster."""

    precision = 32

    def __init__(self, max_steps=0):
        self.descs = [make_desc(N, 0.06, 0.1, wavelength=8e-7, n2=3.2e-23, terms=1)]
        self.max_steps = max_steps
        self.plan, self.adjoint, self.timed = (0, 0), (-1, -1), 0
        self.launches = set()

    def _known(self, *variants):
        if any(not -1 <= v < 2 for v in variants):
            raise L.SsfmError(L.EINVAL, "select", "variant out of range")

    def select_plan(self, n, row, col):
        self._known(row, col)
        self.plan = (row, col)

    def select_adjoint_plan(self, n, row, col):
        self._known(row, col)
        self.adjoint = (row, col)

    def time_passes(self, reps):
        self.timed += 1
        self.launches.add(reps)
        return 2.0 - self.plan[0], 2.0 - self.plan[1], 0.0, 0.0

    def time_adjoint_passes(self, reps):
        self.timed += 1
        self.launches.add(reps)
        return 2.0 - self.adjoint[1], 2.0 - self.adjoint[0]


@pytest.fixture
def cache(tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("SSFM_TUNE_CACHE", str(path))
    monkeypatch.setattr(tuner, "plan_variants", lambda n, precision: (2, 2))
    return path


@pytest.mark.parametrize("row,col", [(6, 6), (0, 0)])
def test_entries_of_other_libraries_are_not_used(cache, row, col):
    """Variants saved with another library (whose indices this one may not have,
    or have for other tiles) are measured anew."""
    name = "none" if not tuner.torch.cuda.is_available() else tuner.torch.cuda.get_device_name(0)
    old = {f"{name}|n={N}|fp32": {"row": row, "col": col, "row_adj": row, "col_adj": col}}
    cache.write_text(json.dumps(old))
    p = _Context(max_steps=4)
    best = tuner.tune(p)[N]
    assert p.timed > 0
    assert (best["row"], best["col"], best["row_adj"], best["col_adj"]) == (1, 1, 1, 1)
    assert p.plan == (1, 1) and p.adjoint == (1, 1)


def test_entries_of_the_same_library_are_used(cache):
    first, second = _Context(max_steps=4), _Context(max_steps=4)
    best = tuner.tune(first)[N]
    again = tuner.tune(second)[N]
    assert second.timed == 0 and second.plan == (1, 1) and second.adjoint == (1, 1)
    assert {k: best[k] for k in ("row", "col", "row_adj", "col_adj")} == \
        {k: again[k] for k in ("row", "col", "row_adj", "col_adj")}


class _Uneven(_Context):
    """Three row and five column variants; rows 1 and columns 2 are not built,
    and the adjoint takes even variants only."""

    def _known(self, *variants):
        pass

    def select_plan(self, n, row, col):
        if row == 1 or col == 2:
            raise L.SsfmError(L.EUNSUPPORTED, "select", "not built")
        super().select_plan(n, row, col)

    def select_adjoint_plan(self, n, row, col):
        if row % 2 == 1 and row > 0 or col % 2 == 1 and col > 0:
            raise L.SsfmError(L.EINVAL, "select", "other lines per workgroup")
        super().select_adjoint_plan(n, row, col)

    def time_passes(self, reps):
        self.timed += 1
        self.launches.add(reps)
        return 10.0 + self.plan[0], 20.0 - self.plan[1], 0.0, 0.0

    def time_adjoint_passes(self, reps):
        self.timed += 1
        self.launches.add(reps)
        return 40.0 + self.adjoint[1], 30.0 - self.adjoint[0]


def test_every_accepted_variant_is_timed_as_itself(cache, monkeypatch):
    """A row and a column variant share a measurement where both are accepted;
    where one is refused, the other is timed beside the base variant."""
    monkeypatch.setattr(tuner, "plan_variants", lambda n, precision: (3, 5))
    p = _Uneven(max_steps=4)
    best = tuner.tune(p, use_cache=False)[N]
    assert best["rows_ms"] == [10.0, 12.0]                      # rows 0, 2
    assert best["cols_ms"] == [20.0, 19.0, 17.0, 16.0]          # columns 0, 1, 3, 4
    assert (best["row"], best["col"]) == (0, 4)
    assert best["rows_adj_ms"] == {0: 30.0, 2: 28.0}
    assert best["cols_adj_ms"] == {0: 40.0, 2: 42.0, 4: 44.0}
    assert (best["row_adj"], best["col_adj"]) == (2, 0)
    assert p.timed == 5 + 3 and p.plan == (0, 4) and p.adjoint == (2, 0)


@pytest.mark.parametrize("reps,launches", [(50, 25), (11, 6), (1, 1)])
def test_a_launch_times_two_factors(cache, reps, launches):
    p = _Context(max_steps=4)
    tuner.tune(p, reps=reps, use_cache=False)
    assert p.launches == {launches}
