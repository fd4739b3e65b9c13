"""List walks that open more cells than a work-group keeps in LDS (5600): they
go through scratch in memory, a part of it for each work-group, which grows
where a walk opens more cells than it holds (32768 at first).  Bit-exact against
the oracle's tree.
"""
import numpy as np
import pytest

from paper_1602_02832_amd import binding as B

from test_gpu_tree import assert_same, build_both

pytestmark = pytest.mark.gpu

# n, n_crit, theta, at least that many groups, nodes and entries
CASES = {
    "more_groups_than_work_groups": (40000, 64, 0.05, 600, 16000, 600 * 30000),
    "one_group_grows_the_scratch": (150000, 10**6, 0.5, 1, 60000, 150000),
    "several_groups_grow_the_scratch": (150000, 30000, 0.03, 4, 60000, 4 * 140000),
}


@pytest.mark.parametrize("name", CASES)
def test_walks_through_memory(oracle, name):
    n, n_crit, theta, groups, nodes, entries = CASES[name]
    print(f"case {name}: n={n} n_crit={n_crit} theta={theta}", flush=True)
    x = np.random.default_rng(21).random((n, 3))
    tree = B.DeviceTree(n_max=n)
    try:
        for seed in (1, 2):   # with the arrays of no build before it, then with its own
            ref, got = build_both(oracle, tree, x, 1, n_crit, theta, seed=seed)
            assert got.n_group >= groups and got.n_node >= nodes and got.n_entries >= entries
            assert_same(ref, got, f"{name} {seed}")
        # a smaller tree on the same object
        ref, got = build_both(oracle, tree, x[:5000], 1, 64, 0.5, seed=3)
        assert_same(ref, got, f"{name} small")
    finally:
        tree.close()
