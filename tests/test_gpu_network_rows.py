"""The FP32 network's rows pass between the lanes of a wavefront through LDS:
each row's energy and input gradient are its own, bit for bit, whatever rows
share its wavefront and wherever it lies among them."""
import numpy as np
import pytest

from paper_2608_14911_amd import inputs
from paper_2608_14911_amd.system import System, lj_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [16, 31, 1000, 70001])
def test_rows_do_not_depend_on_their_neighbours(P):
    box = np.array([9.0] * 3)
    s = System(inputs.random_positions(10, box, seed=1), box, pair={(0, 0): lj_pair(rc=1.12)}, list_cutoff=2.5,
               surrogate=True)
    s.sur_set(0.3 * inputs.mlp_init(seed=7), np.full(32, 0.4), np.full(32, 1.7), "fp32")
    g = inputs.rng(P, 2)
    G = g.uniform(0.0, 2.0, size=(P, 32)).astype(np.float32)
    e, a = (t.cpu().numpy() for t in s.mlp_eval(G))
    order = g.permutation(P)
    e2, a2 = (t.cpu().numpy() for t in s.mlp_eval(G[order]))
    assert np.array_equal(e2, e[order]) and np.array_equal(a2, a[order])
    one = [s.mlp_eval(G[k:k + 1]) for k in (0, P // 2, P - 1)]
    for (ek, ak), k in zip(one, (0, P // 2, P - 1)):
        assert ek.cpu().numpy()[0] == e[k] and np.array_equal(ak.cpu().numpy()[0], a[k])
    s.close()
