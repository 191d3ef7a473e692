"""md_config.block_size in the force kernels beside the FP32 fast ones (FP64,
capped and mixed types, tables, DPD, shear, AdResS, bonds): the size asked for
runs (the FP64 block sums of the observables round differently in blocks of 64
and of 256), forces and trajectories are those of the other size, bit for bit,
and the per-step records are read with the block count that ran."""
import numpy as np
import pytest

from paper_2608_14911_amd import inputs
from paper_2608_14911_amd.system import System, lj_pair

pytestmark = pytest.mark.gpu

N = 3001
KINDS = ("fp64", "capped", "mixture", "tabulated", "dpd", "dpd_shear", "adress", "shear", "fp64_bonded")


def make(kind, block):
    pos, box = inputs.fcc_lattice(10, 0.8442, jitter=0.1, seed=8)
    pos = np.ascontiguousarray(pos[:N])
    vel = inputs.maxwell_boltzmann(N, 1.0, seed=8)
    kw = dict(pair={(0, 0): lj_pair(rc=2.5)}, dt=0.002, skin=0.3, block_size=block, seed=8)
    if kind.startswith("fp64"):
        kw.update(precision="fp64")
    if kind == "fp64_bonded":
        w = inputs.lattice_melt(60, 50, 0.85, seed=5)
        return System(w["pos"], w["box"], inputs.maxwell_boltzmann(3000, 1.0, seed=5),
                      **dict(kw, pair={(0, 0): lj_pair(rc=2 ** (1 / 6))}, bonds=w["bonds"], angles=w["angles"], k_bend=1.5))
    if kind == "capped":
        kw.update(pair={(0, 0): lj_pair(rc=2.5, caprad=0.85)})
    if kind == "mixture":
        rows = {(a, b): lj_pair(rc=2.5 - 0.2 * (a + b)) for a in range(2) for b in range(a, 2)}
        kw.update(pair=rows, types=(np.arange(N) % 2).astype(np.int32), n_types=2, masses=(1.0, 2.0))
    if kind == "tabulated":
        kw.update(table_points=256)
    if kind.startswith("dpd"):
        kw.update(pair={(0, 0): lj_pair(eps=0.0, rc=1.0)}, integrator="dpd", temperature=1.0, gamma=4.5, dpd_rc=1.0)
    if kind in ("dpd_shear", "shear"):
        kw.update(shear_rate=0.3)
        vel[:, 0] += 0.3 * (pos[:, 1] - 0.5 * box[1])
    if kind == "adress":
        kw.update(pair={(0, 0): lj_pair(rc=2.5, caprad=0.85)}, table_points=256, adress=(0.5 * box[0], 0.15 * box[0], 0.2 * box[0]))
    s = System(pos, box, vel, **kw)
    r = np.linspace(0.5, 2.5, 256)
    if kind == "tabulated":
        s.set_pair_table(0, 0, 4.0 * (r ** -12 - r ** -6), 24.0 * (2.0 * r ** -13 - r ** -7), 0.5)
    if kind == "adress":
        s.set_cg_table(0, 0, 2.0 * (1.0 - r / 2.5) ** 2, 1.6 * (1.0 - r / 2.5), 0.5, 2.5)
    return s


SUMS = ("e_pair", "e_bond", "e_angle", "e_kin", "virial")


@pytest.mark.parametrize("kind", KINDS)
def test_asked_size_runs_and_changes_cost_only(kind):
    got = {}
    for block in (0, 64, 256, 128):
        s = make(kind, block)
        f = s.forces()
        s.step(8)
        st, h = s.get_state(), s.history()
        # records of a call's steps agree with the observables of the same state
        s.set_params(block_size=256 if block == 64 else 64)
        s.step(3)
        s.step(4)
        h += s.history()
        assert [x["step"] for x in h] == list(range(15))
        got[block] = (f, st, h, s.get_state())
        s.close()
    f0, st0, h0, end0 = got[0]
    for block, (f, st, h, end) in got.items():
        assert np.array_equal(f, f0) and np.array_equal(st["pos"], st0["pos"]) and np.array_equal(st["vel"], st0["vel"])
        assert np.array_equal(end["pos"], end0["pos"])
        for a, b in zip(h, h0):
            for k in SUMS:
                assert abs(a[k] - b[k]) <= 1e-11 * max(abs(b[k]), 1.0), (block, k)
    same = lambda x, y: all(a[k] == b[k] for a, b in zip(got[x][2][:8], got[y][2][:8]) for k in SUMS)
    # 0 is 64 at this size, and so is a size these kernels do not take
    assert same(0, 64) and same(0, 128) and not same(64, 256)
