"""Rebuilds on one device tree (include/htree_tree.h): a build that finds the
arrays of the one before it queues everything for what they hold, and has to
notice where the counts turn out larger.  Each sequence goes through sizes at
the edges of the kernels' tiles (512 particles, 1024 groups, 1024 keys, 32768 particles' sort) and
through steps that outgrow the cells, the nodes, the groups, the lists' staging
or the entries.  Bit-exact against the oracle's tree, as index work has to be.
"""
import numpy as np
import pytest

from paper_1602_02832_amd import binding as B

pytestmark = pytest.mark.gpu


def uniform(n):
    return np.random.default_rng(n).random((n, 3))


def pairs(n):
    """Particles in pairs 1e-6 apart: each pair has a chain of single-child cells."""
    x = uniform(n)
    x[1::2] = x[: 2 * (n // 2) : 2] + 1e-6
    return x


SEQUENCES = {
    "tile_edges": [(uniform(n), 1, 8, 0.5) for n in (511, 512, 513, 1023, 1024, 1025, 256, 1, 2)],
    "cells_and_nodes": [(uniform(600), 1, 64, 0.6), (pairs(600), 1, 64, 0.6), (pairs(601), 2, 64, 0.6)],
    "groups": [(uniform(3000), 1, 3000, 0.6), (uniform(3000), 1, 1, 0.9), (uniform(2049), 3, 1, 0.9)],
    "sort": [(uniform(n), 1, 512, 0.9) for n in (12345, 32768, 32769)] +
            [(np.floor(3.0 * uniform(n)), 2, 64, 0.7) for n in (1300, 700)],   # 27 keys in all, shared over runs
    "lists": [(uniform(1500), 1, 32, 1.2), (uniform(1500), 1, 32, 0.2), (uniform(1500), 1, 1, 0.0),
              (uniform(1500), 40, 100, 0.5)],
}


@pytest.mark.parametrize("name", SEQUENCES)
def test_rebuilds_match_oracle(oracle, name):
    import torch
    tree = B.DeviceTree(n_max=40000)
    try:
        for k, (x, n_leaf, n_crit, theta) in enumerate(SEQUENCES[name]):
            n = len(x)
            tag = f"{name} step {k}: n={n} n_leaf={n_leaf} n_crit={n_crit} theta={theta}"
            print("case " + tag, flush=True)
            rng = np.random.default_rng(k)
            v, a, j = (rng.standard_normal((n, 3)) for _ in range(3))
            m = rng.random(n) + 0.05
            ref = oracle.Tree(x, v, a, j, m, n_leaf, n_crit, theta)
            for _ in range(2):   # with the last step's arrays, then with its own
                tree.build(*(torch.from_numpy(q).cuda() for q in (x, v, a, j, m)), n_leaf, n_crit, theta)
                got = tree.get()
                assert (got.n_node, got.n_group, got.n_entries) == (ref.n_node, ref.n_group, ref.n_entries), tag
                for f in ("perm", "keys", "node_m", "node_x", "node_v", "node_a", "node_j", "node_level",
                          "node_begin", "node_end", "group_first", "list_off", "entries"):
                    r, g = getattr(ref, f), getattr(got, f)
                    assert r.shape == g.shape and r.tobytes() == g.tobytes(), f"{tag}: {f}"
                assert ref.side == got.side and np.array_equal(ref.lo, got.lo), tag
            ms = tree.phase_ms()
            assert all(q >= 0 for q in ms.values()), ms
    finally:
        tree.close()
