"""The matrix-core list build at the sizes where its segments, chunks and
queues can go wrong: rows equal the per-particle build's, entry for entry."""
import numpy as np
import pytest

from paper_2608_14911_amd import inputs, md
from paper_2608_14911_amd.system import System, lj_pair

pytestmark = pytest.mark.gpu


def rows(pos, box, flags, **kw):
    s = System(pos, box, flags=flags, **kw)
    r = s.neighbors(sort=False)
    s.close()
    return r


# (particles, cells per side, cell factor): the smallest box it takes (4 cells,
# 6 half cells), rows of one, two and many segments, a last tile of one
# particle, chunks of a few candidates (sparse) and of many queue flushes (dense)
@pytest.mark.parametrize("n,side,cf", [(1, 4, 1), (65, 4, 1), (500, 4, 1), (4097, 4, 1), (1000, 6, 2), (3001, 8, 2),
                                       (641, 9, 1), (20000, 11, 1), (6000, 5, 1), (3000, 40, 1)])
@pytest.mark.parametrize("shape", [(1.0, 1.0, 1.0), (1.9, 1.0, 1.3)])
def test_rows_equal_the_per_particle_build(n, side, cf, shape):
    rv = 1.4
    box = np.array(shape) * rv / cf * (side + 0.01)
    pos = inputs.random_positions(n, box, seed=n)
    kw = dict(pair={(0, 0): lj_pair(rc=1.1)}, skin=0.3, cell_factor=cf, nl_capacity=512)
    a = rows(pos, box, md.MD_CFG_NL_TILES, **kw)
    b = rows(pos, box, md.MD_CFG_NL_PER_PARTICLE, **kw)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


# the one-wavefront-per-particle build of small systems: one and several chunks
# of 64 candidates, wrapped ranges, three-cell boxes, the padding's edges, bonds;
# and the one-block sort on both sides of its limit
@pytest.mark.parametrize("n,L,cf", [(1, 4.3, 1), (9, 4.3, 1), (300, 4.3, 1), (2000, 5.7, 1), (1000, 4.3, 2),
                                    (4096, 14.0, 1), (4097, 14.0, 1), (20000, 21.0, 1), (500, 60.0, 1)])
def test_small_builds_equal_the_per_particle_build(n, L, cf):
    pos = inputs.random_positions(n, [L] * 3, seed=n)
    kw = dict(pair={(0, 0): lj_pair(rc=1.1)}, skin=0.3, cell_factor=cf, nl_capacity=512)
    a = rows(pos, [L] * 3, 0, **kw)
    b = rows(pos, [L] * 3, md.MD_CFG_NL_PER_PARTICLE, **kw)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_small_bonded_trajectory_equals_the_per_particle_build():
    w = inputs.lattice_melt(20, 50, 0.85, seed=5)
    got = []
    for flags in (0, md.MD_CFG_NL_PER_PARTICLE):
        s = System(w["pos"], w["box"], inputs.maxwell_boltzmann(1000, 1.0, seed=5), pair={(0, 0): lj_pair(rc=2 ** (1 / 6))},
                   bonds=w["bonds"], angles=w["angles"], k_bend=1.5, dt=0.01, integrator="langevin", gamma=0.5, seed=5,
                   flags=flags)
        s.step(40)
        assert s.observables()["n_rebuilds"] > 4
        got.append(s.get_state())
        s.close()
    assert np.array_equal(got[0]["pos"], got[1]["pos"]) and np.array_equal(got[0]["vel"], got[1]["vel"])


def test_pairs_at_the_list_radius():
    """Pairs placed exactly at the list radius and one ulp to either side are
    decided in FP64 (strictly inside)."""
    rv, L = 1.4, 14.1
    g = inputs.rng(5, inputs.STREAM_POS)
    a = g.uniform(0.0, L, size=(300, 3))
    d = g.standard_normal((300, 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    pos = inputs.wrap_into_box(np.concatenate([a, a + rv * d, a + np.nextafter(rv, 0) * d[::-1]]), [L] * 3)
    kw = dict(pair={(0, 0): lj_pair(rc=1.1)}, skin=0.3, nl_capacity=256)
    x = rows(pos, [L] * 3, md.MD_CFG_NL_TILES, **kw)
    y = rows(pos, [L] * 3, md.MD_CFG_NL_PER_PARTICLE, **kw)
    assert all(np.array_equal(p, q) for p, q in zip(x, y))


@pytest.mark.parametrize("rho,rate", [(3.0, 0.3), (6.0, 0.7)])
def test_sheared_sets_equal_the_per_particle_build(rho, rate):
    """Under shear, after the offset has moved: equal sets (the row order of a
    sheared list is not fixed)."""
    L = 11.0
    n = int(rho * L ** 3)
    pos = inputs.random_positions(n, [L] * 3, seed=3)
    got = []
    for flags in (md.MD_CFG_NL_TILES, md.MD_CFG_NL_PER_PARTICLE):
        s = System(pos, [L] * 3, pair={(0, 0): (0.0, 1.0, 1.0, 0.0, 0.0)}, skin=0.3, dt=0.01, shear_rate=rate,
                   flags=flags, nl_capacity=256)
        st = s.get_state()
        st["step"] = 777
        s.set_state(st, with_build=False)
        got.append(s.neighbors())
        s.close()
    assert all(np.array_equal(p, q) for p, q in zip(*got))
