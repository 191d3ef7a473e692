"""What the autotuner writes down, on the CPU with systems whose cost per step
is given: each trial is recorded under the block size and the build that ran."""
import types

import pytest

from paper_2608_14911_amd import autotune, md
from paper_2608_14911_amd.system import nl_build_flags

FLAGS = {nl_build_flags(b): b for b in ("auto", "tiles", "per_particle")}


class Timed:
    """Cost per step by (build, block size that runs: 0 means 64)."""

    def __init__(self, cost, cf, flags):
        self.cost, self.build = cost, FLAGS[flags]
        self.cfg = types.SimpleNamespace(skin=0.3, cell_factor=cf, block_size=0)

    def set_params(self, **kw):
        for k, v in kw.items():
            setattr(self.cfg, k, v)

    def ms(self):
        return self.cost(self.build, self.cfg.cell_factor, self.cfg.block_size or 64)

    def close(self):
        pass


@pytest.fixture
def fake(monkeypatch):
    monkeypatch.setattr(autotune, "_time_system", lambda s, steps: s.ms())


def cost(build, cf, block):
    return {"auto": 1.0, "tiles": 2.0, "per_particle": 3.0}[build] * cf + 0.1 * (block != 64) + (1.0 if cf == 0 else 0.0)


def test_trials_are_recorded_with_the_size_that_ran(tmp_path, fake):
    path = str(tmp_path / "c.json")
    (cf, build, block, skin), table = autotune.tune_system(lambda c, f: Timed(cost, c, f), 4000, 0.8, 2.5, "lj", path=path)
    for t in table:
        assert t["ms_per_step"] == cost(t["nl_build"], t["cell_factor"], t["block_size"]), t
    assert (cf, build, block, skin) == (1, "tiles", 64, 0.3)
    assert autotune.cached_system_choice("lj", 4000, 0.8, 2.5, path=path) == (1, "tiles", 64, 0.3)


def test_the_automatic_build_can_win_and_is_cached(tmp_path, fake):
    path = str(tmp_path / "c.json")
    builds = autotune.BUILDS + ((0, "auto"),)
    best, table = autotune.tune_system(lambda c, f: Timed(cost, c, f), 2048, 0.8, 2.5, "lj", builds=builds, path=path)
    assert best == (0, "auto", 64, 0.3) and len(table) == 4 + len(autotune.BLOCKS)
    assert autotune.cached_system_choice("lj", 2048, 0.8, 2.5, path=path) == best
    # in a batch too
    m = {"kind": "lj", "pos": md.np.zeros((3000, 3)), "box": [15.5] * 3, "pair": {(0, 0): (1, 1, 2.5, 0, 0)}, "skin": 0.3}
    spent = []

    def timed(ms, steps):
        spent.append(ms[0]["nl_build"])
        return cost(ms[0]["nl_build"], ms[0]["cell_factor"], 64)
    old, autotune.time_batch = autotune.time_batch, timed
    try:
        choice, _ = autotune.tune([m], skins=(0.3,), builds=builds, path=path)
    finally:
        autotune.time_batch = old
    assert spent == ["tiles", "per_particle", "per_particle", "auto"]
    k = autotune.member_key(m)
    assert choice[k] == (0.3, 0, "auto") and autotune.cached_choice([m], path)[0][k] == (0.3, 0, "auto")
    # what was not measured is not written
    def fails(ms, steps):
        raise RuntimeError("too small")
    autotune.time_batch, path2 = fails, str(tmp_path / "d.json")
    try:
        autotune.tune([m], skins=(0.3,), path=path2)
    finally:
        autotune.time_batch = old
    assert autotune.load_cache(path2) == {}
