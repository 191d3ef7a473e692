"""md_plan_list_build on the CPU: the list build a handle of a configuration
runs, at both sides of each rule (host arithmetic only)."""
import ctypes

import pytest

from paper_2608_14911_amd import md

LJ = dict(pair={(0, 0): (1.0, 1.0, 2.5, float("nan"), 0.0)}, skin=0.3)
WCA = dict(pair={(0, 0): (1.0, 1.0, 2.0 ** (1 / 6), float("nan"), 0.0)}, skin=0.4)


def plan(n, rho, box=None, **kw):
    L = [(n / rho) ** (1 / 3)] * 3 if box is None else box
    return md.md_plan_config(md.make_config(n, L, **kw))


@pytest.mark.parametrize("n,rho,kw,build", [
    (1000, 0.85, WCA, "wave"), (20000, 0.8442, LJ, "wave"), (20000, 0.05, LJ, "wave"),
    (20001, 0.8442, LJ, "tiles"), (20001, 0.1, LJ, "per_particle"), (1048576, 0.8442, LJ, "tiles"),
    (2000000, 0.85, WCA, "per_particle"),
    # 5 particles per cell of side rc + skin: 0.2278 at 2.8
    (30000, 0.2270, LJ, "per_particle"), (30000, 0.2285, LJ, "tiles"),
    # very dense small systems: more than 1.2e7 candidates in all
    (19000, 10.0, LJ, "tiles"),
])
def test_automatic_build(n, rho, kw, build):
    p = plan(n, rho, **kw)
    assert p["list_build"] == build
    if build != "wave":
        assert p["nl_build"] == build


@pytest.mark.parametrize("n,rho", [(1000, 0.8442), (6000, 0.8442), (100000, 0.8442), (100000, 0.1)])
def test_sheared_systems_take_tiles_by_density_alone(n, rho):
    p = plan(n, rho, shear_rate=0.1, **LJ)
    dense = rho > 0.2278 and n > 1000       # 1,000 particles: 3 cells per side, no room for tiles
    assert p["list_build"] == p["nl_build"] == ("tiles" if dense else "per_particle")


def test_flags_name_the_build_and_its_limits():
    assert plan(1000, 0.85, flags=md.MD_CFG_NL_TILES, **WCA)["list_build"] == "tiles"
    assert plan(1000, 0.85, flags=md.MD_CFG_NL_PER_PARTICLE, **WCA)["list_build"] == "per_particle"
    # three cells per side: no room for tiles, forced or not
    box = [8.41] * 3
    assert plan(1000, None, box, flags=md.MD_CFG_NL_TILES, **LJ)["list_build"] == "per_particle"
    assert plan(30000, None, box, **LJ)["list_build"] == "per_particle"
    assert plan(30000, None, box, **LJ)["nl_build"] == "per_particle"
    # a box of a different shape: the shortest side counts
    assert plan(30000, None, [8.41, 60.0, 60.0], **LJ)["list_build"] == "per_particle"
    assert plan(30000, None, [11.21, 60.0, 60.0], flags=md.MD_CFG_NL_TILES, **LJ)["list_build"] == "tiles"


def test_arguments():
    b = ctypes.c_int32()
    cfg = md.make_config(1000, [20.0] * 3, **LJ)
    assert md.lib().md_plan_list_build(ctypes.byref(cfg), None) == -1
    assert md.lib().md_plan_list_build(None, ctypes.byref(b)) == -1
    cfg = md.make_config(1000, [6.0] * 3, **LJ)
    with pytest.raises(md.MDError):
        md.md_plan_config(cfg)
    assert md.lib().md_plan_list_build(ctypes.byref(cfg), ctypes.byref(b)) == md.lib().md_plan_config(
        ctypes.byref(cfg), ctypes.byref(md.md_plan()))


@pytest.mark.parametrize("n,rho,kw", [(1048576, 0.8442, LJ), (200000, 3.0, dict(LJ, pair={(0, 0): (1.0, 1.0, 1.0, 0.0, 0.0)})),
                                      (200000, 3.0, dict(LJ, pair={(0, 0): (1.0, 1.0, 1.0, 0.0, 0.0)}, shear_rate=0.1))])
def test_half_cells_are_built_per_particle_unless_tiles_are_asked_for(n, rho, kw):
    assert plan(n, rho, cell_factor=2, **kw)["list_build"] == "per_particle"
    assert plan(n, rho, cell_factor=2, flags=md.MD_CFG_NL_TILES, **kw)["list_build"] == "tiles"
    assert plan(n, rho, **kw)["list_build"] == "tiles"


def test_batch_members_take_tiles_but_for_small_sparse_ones():
    cfg = lambda n, rho, **kw: md.make_config(n, [(n / rho) ** (1 / 3)] * 3, **kw)
    skin5 = dict(WCA, skin=0.5)
    cases = [(cfg(500, 0.85, **skin5), "per_particle"), (cfg(2048, 0.85, **skin5), "per_particle"),
             (cfg(2049, 0.85, **skin5), "tiles"), (cfg(250000, 0.85, **skin5), "tiles"),
             (cfg(500, 0.85, flags=md.MD_CFG_NL_TILES, **skin5), "tiles"),
             (cfg(30000, 0.85, flags=md.MD_CFG_NL_PER_PARTICLE, **skin5), "per_particle"),
             (cfg(1000, 0.8, **LJ), "per_particle"),     # 3 cells per side
             (cfg(1500, 0.8, **LJ), "tiles"), (cfg(30000, 0.8, **LJ), "tiles"),
             (cfg(30000, 0.8, cell_factor=2, **LJ), "per_particle")]
    assert md.md_batch_plan_list_build([c for c, _ in cases]) == [b for _, b in cases]
    for c, b in cases:      # a member's build does not depend on the others
        assert md.md_batch_plan_list_build([c]) == [b]
    with pytest.raises(md.MDError):
        md.md_batch_plan_list_build([])
