"""Edges of the force launch's choices: sums of split tiles by the tile's last
item up to 16384 partial slots and by a launch of their own above, tiles of up
to 64 slots alone and with the two-slot tiles of 128 and 256, and the device
loop and the state upload at small and odd particle numbers.  Forces against
the oracle at the tolerances of parity_util; where two routes sum in the same
order, bit for bit.
"""
import numpy as np
import pytest

from paper_1602_02832_amd import binding as B
from paper_1602_02832_amd import driver
from paper_1602_02832_amd import workloads as W

from parity_util import assert_close, oracle_list_force, say

pytestmark = pytest.mark.gpu


def context(prec, n, tree=None, eps2=1e-4):
    node_max, group_max, list_max = (16, 1, 16) if tree is None else (2 * n, n, 2 * tree.n_entries)
    return B.Context(n_max=n, node_max=node_max, group_max=group_max, list_max=list_max, active_max=n, eps2=eps2,
                     precision=prec)


# 12 rounds of 256 entries: at most 12 splits a tile, so 16380 slots (folded) and 16392 (a launch)
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("k", [1, 64, 65, 127, 128, 129, 192, 255, 257, 1365, 1366, 3000])
def test_direct_splits_match_oracle(oracle, prec, k):
    say(f"direct splits {prec} n_active={k}")
    n = 3000
    x, v, _ = W.plummer(n, 61)
    m = W.salpeter_masses(n, 62)
    z = np.zeros((n, 3))
    c = context(prec, n)
    c.set_j_particles(0.25, m, x, v, z, z)
    c.set_nodes(0.0, np.zeros(0), z[:0], z[:0], z[:0], z[:0])
    c.set_tuning(12, 1 << 20)
    c.predict(0.25)
    ids = np.sort(np.random.default_rng(k).choice(n, k, replace=False)).astype(np.int32)
    mj = m if prec == "fp64" else m.astype(np.float32).astype(np.float64)
    assert_close(f"direct n_active={k}", prec, c.force_direct(ids), oracle.force_direct(ids, x, v, mj, 1e-4))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("target", [1, 2048, 6000, 1 << 20])
def test_list_splits_match_oracle_and_the_captured_step(oracle, prec, target):
    """With many items asked for, the split sums pass 16384 slots and get a
    launch; the captured step always sums in the force launch."""
    import torch
    say(f"list splits {prec} target={target}")
    n, t = 6000, 0.25 + 1.0 / 64
    x, v, m = W.plummer(n, 71)
    z = np.zeros((n, 3))
    tr = oracle.Tree(x, v, z, z, m, 1, 700, 0.5)
    x, v, m = x[tr.perm], v[tr.perm], m[tr.perm]
    t0, a, j = W.random_block_state(n, 72, 0.25)
    if prec == "mixed":   # what the form stores in FP32 is given exactly
        f32 = lambda q: q.astype(np.float32).astype(np.float64)  # noqa: E731
        a, j, m = f32(a), f32(j), f32(m)
        tr.node_m, tr.node_a, tr.node_j = f32(tr.node_m), f32(tr.node_a), f32(tr.node_j)
    ctxs = []
    for _ in range(2):
        c = context(prec, n, tr)
        c.set_j_particles(t0, m, x, v, a, j)
        c.set_nodes(0.0, tr.node_m, tr.node_x, tr.node_v, tr.node_a, tr.node_j)
        c.set_interaction_lists(tr.group_first, tr.list_off, tr.entries)
        c.set_tuning(12, target)
        ctxs.append(c)
    rng = np.random.default_rng(73)
    for k in (1, 40, 700, n):
        act = np.sort(rng.choice(n, k, replace=False)).astype(np.int32)
        outs = [tuple(torch.full(s, float("nan"), dtype=torch.float64, device="cuda") for s in ((k, 3), (k, 3), (k,)))
                for _ in range(2)]
        ctxs[0].step_async(None, t, act, *outs[0])
        ctxs[1].step_graph(None, t, act, *outs[1])
        for c in ctxs:
            c.sync()
        for p, q in zip(*outs):
            assert torch.equal(p, q), (target, k)
        want = oracle_list_force(oracle, t, act, t0, m, x, v, a, j, tr, 1e-4)
        assert_close(f"list splits n_active={k}", prec, tuple(p.cpu().numpy() for p in outs[0]), want)


@pytest.mark.parametrize("n", [2, 65, 257, 1025, 2000])
def test_device_loop_small_sets_equal_step_by_step(n):
    """The loop's planner and corrector with one, a few and all particles due."""
    say(f"device loop n={n}")
    x, v, m = W.plummer(n, 80 + n)
    sims = [driver.Simulation(x, v, m, eps2=1e-3, dt_tree=1.0 / 64, eta=0.1, theta=0.5, n_crit=32, precision="mixed",
                              resident=True, device_tree=True, device_loop=d) for d in (False, True)]
    for s in sims:
        s.run(2.0 / 64)
        s.sync_state()
    assert sims[0].n_block_steps == sims[1].n_block_steps and sims[0].t == sims[1].t
    for f in ("x", "v", "a", "j", "t0", "dt", "pot"):
        assert np.array_equal(getattr(sims[0], f), getattr(sims[1], f)), f
    for s in sims:
        s.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_state_upload_writes_the_records(prec):
    """ht_state_set sends the state once and writes the j-records from it on the
    device: the forces are those of ht_set_j_particles, also after a second,
    smaller state."""
    say(f"state upload {prec}")
    rng = np.random.default_rng(5)
    both = [context(prec, 700) for _ in range(2)]
    both[0].state_enable()
    for n in (700, 257, 1):
        t0, dt, m = np.full(n, 0.25), np.full(n, 2.0 ** -7), rng.random(n) + 0.1
        x, v, a, j = rng.standard_normal((4, n, 3))
        both[0].state_set(t0, dt, m, x, v, a, j)
        both[1].set_j_particles(t0, m, x, v, a, j)
        for got, sent in zip(both[0].state_get(), (t0, dt, x, v, a, j)):
            assert np.array_equal(got, sent)
        out = []
        for c in both:
            c.set_nodes(0.25, np.zeros(0), *(np.zeros((0, 3)) for _ in range(4)))
            c.predict(0.25 + 2.0 ** -8)
            out.append(c.force_direct(np.arange(n, dtype=np.int32)))
        for p, q in zip(*out):
            assert np.array_equal(p, q), n
