"""Cached autotuner choices on the CPU: an entry of the cache serves every
system of its bucket and all smaller ones, so what the box of a member cannot
hold is left to half-cutoff cells or to the library's automatic choice."""
import json
import math

import numpy as np
import pytest

from paper_2608_14911_amd import autotune, md
from paper_2608_14911_amd.system import lj_pair, nl_build_flags


def member(n, rho, kind="lj", skin=0.3):
    L = (n / rho) ** (1.0 / 3.0)
    rc = 2.5 if kind == "lj" else 2.0 ** (1.0 / 6.0)
    return {"kind": kind, "pos": np.zeros((n, 3)), "box": np.array([L] * 3), "pair": {(0, 0): lj_pair(rc=rc)},
            "skin": skin}


def config(m):
    return md.make_config(m["pos"].shape[0], m["box"], pair=m["pair"], skin=m["skin"],
                          cell_factor=m.get("cell_factor", 0), flags=nl_build_flags(m.get("nl_build", "auto")))


@pytest.mark.parametrize("n", [300, 350, 400, 500, 700, 1000, 1400, 2047, 2048, 5000, 40000])
@pytest.mark.parametrize("rho", [0.70, 0.75, 0.80, 0.85])
def test_cached_choices_are_accepted(n, rho):
    m = member(n, rho)
    assert "gfx950|lj|n%d|rho%s|rc2.5000" % (autotune.n_bucket(n), autotune.rho_bucket(rho)) in autotune.load_cache()
    a, = autotune.apply([m], autotune.cached_choice([m])[0])
    # a box of 2.5 list radii (5 half cells) is what the library can take at all
    assert m["box"][0] > 2.5 * 2.8
    plan = md.md_plan_config(config(a))
    assert md.md_batch_workspace_bytes([config(a)]) > 0
    cells = int(m["box"][0] / 2.8)
    if cells < 4:   # no room for the tile build of the entry: half cells, one particle per lane
        assert plan["cell_factor"] == 2 and plan["nl_build"] == "per_particle"
    else:
        assert plan["cell_factor"] == 1 and plan["cells"] == [cells] * 3


def test_cached_entry_that_no_cells_hold_leaves_the_member_as_it_was(tmp_path):
    """An entry's larger skin must not make a box too small."""
    m = member(400, 0.85, skin=0.3)     # 7.78: 5 half cells at 2.8, 4 at 3.2
    path = str(tmp_path / "c.json")
    json.dump({autotune.member_key(m): {"skin": 0.7, "cell_factor": 1, "nl_build": "per_particle", "source": "batch"}},
              open(path, "w"))
    a, = autotune.apply([m], autotune.cached_choice([m], path)[0])
    assert (a["skin"], a["cell_factor"], a["nl_build"]) == (0.3, 0, "auto")
    assert md.md_plan_config(config(a))["cell_factor"] == 2


def test_tuned_choices_stand():
    """tune() measured its choice on the members: apply() takes it as it is."""
    m = member(1000, 0.8)
    k = autotune.member_key(m)
    a, = autotune.apply([m], {k: (0.3, 1, "tiles")})
    assert (a["skin"], a["cell_factor"], a["nl_build"]) == (0.3, 1, "tiles")
    kg = member(500, 0.85, "kg", 0.4)
    b, = autotune.apply([kg], autotune.cached_choice([kg])[0])
    assert (b["skin"], b["cell_factor"], b["nl_build"]) == (0.5, 1, "auto")
    assert math.floor(b["box"][0] / (2.0 ** (1.0 / 6.0) + 0.5)) == 5
