"""Per-step records written by the next step's kernel: the same, bit for bit,
as when every step is a call of its own (each record then ends its call)."""
import numpy as np
import pytest

from paper_2608_14911_amd import inputs, md
from paper_2608_14911_amd.system import Batch, System, lj_pair

pytestmark = pytest.mark.gpu


def system(kind, block):
    if kind == "lj":
        w = inputs.workload_lj(ncell=6, seed=3)
        return System(w["pos"], w["box"], w["vel"], pair={(0, 0): lj_pair(rc=2.5)}, block_size=block)
    if kind == "fp64":
        w = inputs.workload_lj(ncell=6, seed=3)
        return System(w["pos"], w["box"], w["vel"], pair={(0, 0): lj_pair(rc=2.5)}, precision="fp64")
    if kind == "capped":
        w = inputs.workload_lj(ncell=6, seed=3)
        return System(w["pos"], w["box"], w["vel"], pair={(0, 0): lj_pair(rc=2.5, caprad=0.8)})
    if kind == "dpd":
        box = np.array([7.0] * 3)
        pos = inputs.random_positions(1000, box, seed=4)
        return System(pos, box, pair={(0, 0): (0.0, 1.0, 1.0, 0.0, 0.0)}, dt=0.01, integrator="dpd", gamma=4.5,
                      temperature=1.0, dpd_rc=1.0, shear_rate=0.2, seed=4)
    w = inputs.lattice_melt(20, 50, 0.85, seed=5)
    s = System(w["pos"], w["box"], inputs.maxwell_boltzmann(1000, 1.0, seed=5), pair={(0, 0): lj_pair(rc=2.0 ** (1 / 6))},
               bonds=w["bonds"], angles=w["angles"], k_bend=1.5, dt=0.01, integrator="langevin", gamma=0.5, seed=5,
               list_cutoff=2.5 if kind == "surrogate" else 0.0, surrogate=kind == "surrogate")
    if kind == "surrogate":
        s.sur_set(0.1 * inputs.mlp_init(seed=6), np.zeros(32), np.ones(32), "bf16")
        s.set_pair_mode("surrogate")
    return s


KEYS = ("step", "e_pair", "e_bond", "e_angle", "e_kin", "virial", "n_rebuilds", "status_flags", "nl_max_count")


@pytest.mark.parametrize("kind,block", [("lj", 64), ("lj", 256), ("lj", 512), ("fp64", 0), ("capped", 0), ("dpd", 0),
                                        ("melt", 0), ("surrogate", 0)])
def test_records_of_one_call_and_of_many(kind, block):
    got = []
    for calls in ([25], [1] * 25, [3, 4, 1, 17]):
        s = system(kind, block)
        for n in calls:
            s.step(n)
        got.append((s.history(), s.get_state()))
        s.close()
    (h0, s0) = got[0]
    assert [r["step"] for r in h0] == list(range(25))
    assert h0[-1]["n_rebuilds"] > h0[0]["n_rebuilds"] or kind in ("lj", "fp64", "capped")
    for h, s in got[1:]:
        assert np.array_equal(s["pos"], s0["pos"]) and np.array_equal(s["vel"], s0["vel"])
        for a, b in zip(h, h0):
            assert all(a[k] == b[k] for k in KEYS)


def test_tensor_records():
    got = []
    for calls in ([9], [1] * 9):
        w = inputs.workload_lj(ncell=6, seed=3)
        s = System(w["pos"], w["box"], w["vel"], pair={(0, 0): lj_pair(rc=2.5)}, flags=md.MD_CFG_VIRIAL_TENSOR)
        for n in calls:
            s.step(n)
        got.append(s.history())
        s.close()
    for a, b in zip(*got):
        assert np.array_equal(a["virial_tensor"], b["virial_tensor"]) and np.any(a["virial_tensor"] != 0)
        assert abs(a["virial_tensor"][:3].sum() - a["virial"]) <= 1e-5 * abs(a["virial"]) + 1e-3


def test_batch_observables_after_one_call_and_many():
    reps = inputs.batch_replicas(4, seed=9, n_min=2048, n_max=4096)
    reps = [r for r in reps if r["kind"] == "lj"]
    got = []
    for calls in ([12], [1] * 12):
        b = Batch(reps)
        for n in calls:
            b.step(n)
        got.append((b.observables(), [b.get_state(k) for k in range(len(reps))]))
        b.close()
    (o0, s0), (o1, s1) = got
    for k in range(len(reps)):
        assert s0[k]["step"] == s1[k]["step"] == 12
        assert np.array_equal(s0[k]["pos"], s1[k]["pos"]) and o0[k]["e_total"] == o1[k]["e_total"]
