"""ht_set_tuning's item target: the tiles of a call with too little work are
split into list ranges until it has about that many items."""
import numpy as np
import pytest

from paper_1602_02832_amd import binding as B
from paper_1602_02832_amd import workloads as W

from parity_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("target,items", [(1, 1), (2, 2), (4, 4), (8, 6), (16, 12), (2048, 12)])
def test_a_tile_is_split_into_the_items_asked_for(target, items):
    """One tile of 256 slots over 3000 particles: 12 rounds, which the splits share in whole rounds."""
    say(f"item target {target}")
    n = 3000
    x, v, m = W.plummer(n, 61)
    z = np.zeros((n, 3))
    c = B.Context(n_max=n, node_max=16, group_max=1, list_max=16, active_max=n, eps2=1e-4, precision="fp64")
    c.set_j_particles(np.zeros(n), m, x, v, z, z)
    c.set_nodes(0.0, np.zeros(0), z[:0], z[:0], z[:0], z[:0])
    c.set_tuning(12, target)
    c.predict(0.0)
    c.force_direct(np.arange(256, dtype=np.int32))
    assert c.last_stats() == (256 * n, items)
    c.close()
