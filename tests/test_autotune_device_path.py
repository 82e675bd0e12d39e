"""The tuners where they measure filters (a stand-in context and clock): only what
differs is measured, only what was measured is set."""
import os

import pytest

from paper_1903_10959_amd import autotune as AT


class _X:
    def __init__(self, ncols):
        self.shape = (1000, ncols)


class _Ctx:
    """A context whose filter takes cost[variant] seconds per step."""

    def __init__(self, p, n_el, cost, clock):
        self.p, self.n_el, self.cost, self.clock = p, n_el, cost, clock
        self.tile_variant, self.cells_per_tile, self.filters, self.widths = -1, 2, [], []

    def set_tile_variant(self, v):
        self.tile_variant = v

    def set_cells_per_tile(self, v):
        self.cells_per_tile = v

    def chebyshev_filter(self, X, degree, a, b, a0, prec="fp64", block_width=0):
        self.filters.append(self.tile_variant)
        self.widths.append(block_width)
        self.clock[0] += degree * self.cost[self.tile_variant]


@pytest.fixture
def clock(monkeypatch):
    t = [0.0]
    monkeypatch.setattr(AT.time, "perf_counter", lambda: t[0])
    return t


@pytest.mark.parametrize("p,prec", [(5, "fp32"), (6, "fp32"), (4, "bf16"), (6, "fp64"), (7, "fp64"), (2, "fp64"), (9, "fp64")])
def test_one_tile_is_not_measured_and_changes_nothing(tmp_path, clock, p, prec):
    c = _Ctx(p, 8, {-1: 3.0, 0: 1.0, 1: 2.0}, clock)
    c.set_tile_variant(1)                            # set for another precision
    path = str(tmp_path / "c.json")
    assert AT.tune_tile_variant(c, _X(64), (1.0, 9.0, -1.0), prec, arch="gfx950", cache_path=path) == -1
    assert c.filters == [] and c.tile_variant == 1 and not os.path.exists(path)


@pytest.mark.parametrize("cost,best", [({-1: 1.0, 0: 1.0, 1: 2.0}, -1), ({-1: 1.02, 0: 1.0, 1: 2.0}, -1),
                                       ({-1: 1.5, 0: 1.6, 1: 1.0}, 1), ({-1: 1.5, 0: 1.0, 1: 1.6}, 0)])
def test_two_tiles_against_the_librarys_choice(tmp_path, clock, cost, best):
    path = str(tmp_path / "c.json")
    c = _Ctx(5, 8, cost, clock)
    assert AT.tune_tile_variant(c, _X(64), (1.0, 9.0, -1.0), "fp64", arch="gfx950", cache_path=path) == best
    assert c.tile_variant == best and set(c.filters) == {-1, 0, 1} and set(c.widths) == {64}
    n = len(c.filters)
    assert AT.tune_tile_variant(c, _X(64), (1.0, 9.0, -1.0), "fp64", arch="gfx950", cache_path=path) == best
    assert len(c.filters) == n                       # cached
    for d, x in ((_Ctx(5, 9, cost, clock), _X(64)), (_Ctx(5, 8, cost, clock), _X(65))):
        AT.tune_tile_variant(d, x, (1.0, 9.0, -1.0), "fp64", arch="gfx950", cache_path=path)
        assert d.filters                             # another mesh, another width: measured again


def test_an_entry_of_other_tiles_is_not_used_and_a_trial_restores_the_setting(tmp_path, clock):
    path = str(tmp_path / "c.json")
    AT.save_cache({"tile|gfx950|p5|fp64": {"variant": 0}}, path)
    c = _Ctx(5, 8, {-1: 1.5, 0: 1.6, 1: 1.0}, clock)
    c.set_tile_variant(0)
    assert AT.tune_tile_variant(c, _X(64), (1.0, 9.0, -1.0), "fp64", arch="gfx950", cache_path=path, apply=False) == 1
    assert c.tile_variant == 0


def test_cells_per_tile_is_not_measured(tmp_path, clock):
    path = str(tmp_path / "c.json")
    c = _Ctx(5, 8, {-1: 1.0}, clock)
    assert AT.tune_cells_per_tile(c, _X(24), (1.0, 9.0, -1.0), "fp32", arch="gfx950", cache_path=path) == 0
    assert c.filters == [] and c.cells_per_tile == 0 and not os.path.exists(path)
