"""The step kernel of an AdResS fluid of one particle type, in blocks of 64 and
of 256 threads, at sizes that leave the last wavefront and the last batch of a
row ragged, with a tabulated pair in place of the LJ one and with bonds, against
the FP64 oracle: forces within 1e-5 per particle of the sum of the atomistic,
coarse-grained and bonded force magnitudes, energies and the virial within 1e-5
of theirs.  The fluid is dense, so no particle's scale is that of a lone pair
at the cutoff.
"""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_forces_close, banner, oracle_pp
from paper_2608_14911_amd import inputs
from paper_2608_14911_amd.system import System, lj_pair

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.mark.parametrize("cells,drop,block,table,bonded", [
    (6, 0, 64, False, False), (6, 41, 256, True, False), (8, 3, 256, False, True), (6, 1, 64, True, True)])
def test_adress_step_kernel_forces(cells, drop, block, table, bonded):
    banner("AdResS step: %d cells less %d, blocks of %d, table %d, bonds %d" % (cells, drop, block, table, bonded))
    pos, box = inputs.fcc_lattice(cells, 0.8442, jitter=0.15, seed=13)
    pos = np.ascontiguousarray(pos[:pos.shape[0] - drop])
    n = pos.shape[0]
    zone = (0.5 * box[0], 0.15 * box[0], 0.2 * box[0])
    kw, okw = {}, {}
    if bonded:   # each particle to its nearest free neighbour
        bonds, free = [], np.ones(n, bool)
        for k in range(n):
            if not free[k]:
                continue
            d = pos - pos[k]
            d -= box * np.round(d / box)
            r2 = (d * d).sum(1)
            r2[k] = 1e9
            r2[~free] = 1e9
            j = int(np.argmin(r2))
            if r2[j] < 1.6 ** 2:
                bonds.append((k, j))
                free[k] = free[j] = False
        kw = {"bonds": np.array(bonds, dtype=np.int32), "fene_K": 20.0, "fene_R0": 2.0}
        okw = dict(kw)
    s = System(pos, box, pair={(0, 0): lj_pair(rc=2.5)}, skin=0.3, table_points=512, adress=zone, block_size=block, **kw)
    r = np.linspace(0.0, 2.0, 500)
    cg = (7.5 * (1.0 - r / 2.0) ** 2, 7.5 * (1.0 - r / 2.0))
    s.set_cg_table(0, 0, cg[0], cg[1], 0.0, 2.0)
    at = None
    if table:
        ra = np.linspace(0.2, 2.5, 500)
        at = (0.2, 4.0 * (2.5 - ra) ** 2, 8.0 * (2.5 - ra))
        s.set_pair_table(0, 0, at[1], at[2], at[0])
    Fg, o = s.forces(), s.observables()
    s.close()
    pair = {} if at is None else {"pair": {(0, 0): at}}
    tabs = oracle.tables(adress=zone, cg={(0, 0): (0.0, 2.0) + cg}, **pair)
    Fo, _, oo = oracle.forces_ext(pos, box, oracle_pp(rc=2.5), tabs=tabs, **okw)
    _, _, oa = oracle.forces_ext(pos, box, oracle_pp(rc=2.5), want_fscale=True,
                                 tabs=oracle.tables(**pair) if pair else None, **okw)
    _, _, oc = oracle.forces_ext(pos, box, oracle_pp(rc=2.0), want_fscale=True,
                                 tabs=oracle.tables(pair={(0, 0): (0.0,) + cg}))
    assert_forces_close(Fg, Fo, oa["fscale"] + oc["fscale"], TOL, "AdResS step kernel")
    for k in ("e_pair", "e_bond"):
        assert abs(o[k] - oo[k]) <= TOL * abs(oo[k]), k
    assert abs(o["virial"] - oo["virial"]) <= TOL * oo["virial_abs"]
