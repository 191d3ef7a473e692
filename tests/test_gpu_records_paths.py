"""Per-step records on the paths that lay their partial sums out differently:
the surrogate's FP32 and BF16 forms, with more energy columns than the FP32
network has blocks (256) and with fewer, the timed stages, and batches.  The
same bits whether a record is written by the next step's kernel, at a call's
end or by a timed step, and the energies of md_observables at the same state."""
import numpy as np
import pytest

from paper_2608_14911_amd import inputs
from paper_2608_14911_amd.system import Batch, System, lj_pair

pytestmark = pytest.mark.gpu

KEYS = ("step", "e_pair", "e_bond", "e_angle", "e_kin", "virial", "n_rebuilds", "status_flags", "nl_max_count")


def surrogate(chains, form):
    w = inputs.lattice_melt(chains, 50, 0.85, seed=5)
    n = 50 * chains
    s = System(w["pos"], w["box"], inputs.maxwell_boltzmann(n, 1.0, seed=5), pair={(0, 0): lj_pair(rc=2.0 ** (1 / 6))},
               bonds=w["bonds"], angles=w["angles"], k_bend=1.5, dt=0.005, integrator="langevin", gamma=0.5, seed=5,
               skin=0.3, list_cutoff=2.5, surrogate=True)
    s.sur_set(0.1 * inputs.mlp_init(seed=6), np.zeros(32), np.ones(32), form)
    s.set_pair_mode("surrogate")
    return s


def fluid(seed=3):
    w = inputs.workload_lj(ncell=6, seed=seed)
    return w


@pytest.mark.parametrize("form", ["fp32", "bf16"])
@pytest.mark.parametrize("chains", [20, 1400])
def test_surrogate_records(chains, form):
    print("surrogate records: %d chains, %s" % (chains, form), flush=True)
    got = []
    for calls in ([9], [1] * 9, [2, 3, 1, 3]):
        s = surrogate(chains, form)
        o = s.observables()
        for n in calls:
            s.step(n)
        h, st = s.history(), s.get_state()
        last = s.observables()
        s.step(2)
        h += s.history()
        got.append((h, st))
        s.close()
        assert [r["step"] for r in h] == list(range(11))
        # the sums of a step and of md_observables at its positions: the same
        # terms, the pair energy's in the same columns
        for k in ("e_pair", "e_bond", "e_angle", "virial"):
            scale = 1e-9 * (abs(o[k]) + abs(o["e_pair"]) + abs(o["e_bond"]))
            assert abs(h[0][k] - o[k]) <= scale and abs(h[9][k] - last[k]) <= scale, k
    for h, st in got[1:]:
        assert np.array_equal(st["pos"], got[0][1]["pos"])
        for a, b in zip(h, got[0][0]):
            assert all(a[k] == b[k] for k in KEYS)


@pytest.mark.parametrize("kind", ["lj", "surrogate"])
def test_timed_steps_write_the_same_records(kind):
    got = []
    for timed in (False, True, None):
        if kind == "lj":
            w = fluid()
            s = System(w["pos"], w["box"], w["vel"], pair={(0, 0): lj_pair(rc=2.5)})
        else:
            s = surrogate(20, "fp32")
        for k, n in enumerate((7, 1, 8)):
            s.timing(timed if timed is not None else k == 1)
            s.step(n)
        h = s.history()
        got.append((h, s.get_state()))
        s.close()
        assert [r["step"] for r in h] == list(range(16))
    for h, st in got[1:]:
        assert np.array_equal(st["vel"], got[0][1]["vel"])
        for a, b in zip(h, got[0][0]):
            assert all(a[k] == b[k] for k in KEYS)


def test_batch_steps_count_alike_however_they_are_called():
    """Steps, rebuild counts and observables of batches stepped in one call, one
    by one, timed, and read member by member in between."""
    reps = [dict(fluid(k), pair={(0, 0): lj_pair(rc=2.5)}, dt=0.005, skin=0.3, seed=k) for k in (3, 4)]
    w = inputs.lattice_melt(20, 50, 0.85, seed=5)
    reps.append({"pos": w["pos"], "box": w["box"], "bonds": w["bonds"], "angles": w["angles"], "k_bend": 1.5, "seed": 5,
                 "vel": inputs.maxwell_boltzmann(1000, 1.0, seed=5), "pair": {(0, 0): lj_pair(rc=2 ** (1 / 6))}, "dt": 0.01,
                 "skin": 0.3, "integrator": "langevin", "temperature": 1.0, "gamma": 0.5})
    got = []
    for how in ("once", "single", "timed", "read"):
        b = Batch(reps)
        for n in ([30] if how in ("once", "timed") else [1] * 30 if how == "single" else [5, 1, 10, 14]):
            b.timing(how == "timed")
            b.step(n)
            if how == "read":
                assert b.get_state(1)["step"] == b.get_state(2)["step"]
                b.observables()
        got.append((b.observables(), [b.get_state(k) for k in range(3)]))
        b.close()
    for o, st in got:
        for k in range(3):
            assert o[k]["step"] == st[k]["step"] == 30
            assert np.array_equal(st[k]["pos"], got[0][1][k]["pos"]) and np.array_equal(st[k]["vel"], got[0][1][k]["vel"])
            assert o[k]["e_total"] == got[0][0][k]["e_total"] and o[k]["n_rebuilds"] == got[0][0][k]["n_rebuilds"]
    assert got[0][0][2]["n_rebuilds"] > 3
