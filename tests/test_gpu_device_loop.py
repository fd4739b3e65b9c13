"""Edges of the device loops (ht_dev_run, ht_batch_dev_run) where the selection
launch takes another way.  Bit for bit against the same steps taken one at a
time.
"""
import numpy as np
import pytest

from paper_1602_02832_amd import binding as B
from paper_1602_02832_amd import driver
from paper_1602_02832_amd import engine as E
from paper_1602_02832_amd import workloads as W

from parity_util import say

pytestmark = pytest.mark.gpu

FIELDS = ("t0", "dt", "x", "v", "a", "j", "pot")


def against_single_steps(n, chunk, cases):
    """Three steps of the loop, in which the given particles are due first: for
    each case, (block, how many of its particles) pairs, blocks of chunk particles."""
    top = 1.0 / 256
    x, v, m = W.plummer(n, 91)
    sim = driver.Simulation(x, v, m, eps2=1e-6, dt_tree=top, eta=0.1, theta=0.6, n_crit=1024, precision="mixed",
                            resident=True)
    ctx = sim.ctx
    t0 = np.zeros(n)
    for due in cases:
        dt = np.full(n, top)
        for b, k in due:
            size = min(chunk, n - b * chunk)
            first = b * chunk + (size - k) // 2
            dt[first:first + k] = top * 2.0 ** -20      # the first steps double: all of them stay due together
        state = (t0, dt, sim.m, sim.x, sim.v, sim.a, sim.j, sim.pot)
        ctx.state_set(*state)
        times, count = [], 0
        for _ in range(3):
            t, active = ctx.dev_next_block()
            ctx.dev_step(0.1, top)
            times.append(t)
            count += active.size
        want = ctx.state_get()
        ctx.state_set(*state)
        steps, t_last, psteps = ctx.dev_run(0.1, top, top / 2, 3)
        got = ctx.state_get()
        assert (steps, t_last, psteps) == (3, times[-1], count), due
        assert count >= sum(k for _, k in due), due
        for f, p, q in zip(FIELDS, got, want):
            assert np.array_equal(p, q), (due, f)
    sim.close()


def test_one_block_due_alone_with_more_particles_than_a_work_group():
    """Above 524288 particles a scheduler block holds more than the 512 that the
    planner keeps in LDS.  Where such a block is the only one due, the planner
    reads its count and particles from memory, written in the same work-group."""
    say("device loop: one block of up to 547 particles due alone")
    n = 560000
    assert (n + 1023) // 1024 == 547                    # particles of a scheduler block
    # the counts of one case are not those of the next
    against_single_steps(n, 547, ([(900, 100)], [(900, 512)], [(900, 513)], [(900, 547)], [(3, 547)],
                                  [(900, 530), (901, 547)], [(1022, 547)]))


def test_last_block_with_one_particle():
    """The planner loads the first particles of every due block with the counts;
    the last block may have fewer."""
    say("device loop: last block of one particle")
    n = 600 * 512 + 1
    against_single_steps(n, 512, ([(600, 1)], [(0, 3), (600, 1)], [(599, 512), (600, 1)], [(599, 4), (600, 1)]))


def resident(n, seed, stream, **kw):
    x, v, m = W.plummer(n, seed)
    return driver.Simulation(x, v, m, eps2=1e-4, dt_tree=1.0 / 64, eta=0.02, theta=0.5, n_crit=64, precision="mixed",
                             resident=True, stream=stream.cuda_stream, **kw)


def batch_of(k, stream):
    return B.Batch(stream=stream.cuda_stream, max_clusters=k, max_items=1 << 15, max_active=1 << 13, max_rows=1 << 13)


def test_batch_of_one_reports_its_engine_steps():
    """A wall time for every engine step, also where the batch holds one context."""
    import torch
    say("batched device loop: one context")
    stream = torch.cuda.Stream()
    alone, batched = (resident(1500, 92, stream) for _ in range(2))
    batch = batch_of(1, stream)
    handles = np.array([batched.ctx.handle.value], np.uint64)
    for most in (1, 7, 40):
        k, t, p = alone.ctx.dev_run(0.02, 1.0 / 64, 1.0 / 64, most)
        steps, t_last, psteps, pairs, step_ms = batch.dev_run(handles, [0.02], [1.0 / 64], [1.0 / 64], [most], 64)
        assert (steps[0], t_last[0], psteps[0]) == (k, t, p) and pairs[0] == alone.ctx.last_stats()[0]
        assert len(step_ms) == k > 0 and (step_ms > 0.0).all()
    for q, w in zip(batched.ctx.state_get(), alone.ctx.state_get()):
        assert np.array_equal(q, w)
    for s in (alone, batched, batch):
        s.close()


def test_engine_with_one_cluster_counts_its_steps():
    """The engine's step counts and times, of which its percentiles are taken."""
    say("engine: device loop with one cluster")
    eng = E.Engine(max_clusters=2, max_active=1 << 13, max_items=1 << 15, max_rows=1 << 13, resident=True,
                   device_tree=True, tree_n_max=2000, device_loop=True, loop_steps=16)
    c = eng.new_cluster(E.RunSpec(key=0, n=1200, seed=93, steps=40, n_crit=64))
    eng.add(c)
    while not c.done:
        eng.step()
    eng.drain()
    assert c.steps_done == 40 and eng.engine_steps == 40 and len(eng.step_ms) == 40
    eng.close()


@pytest.mark.parametrize("first", [True, False])
def test_context_that_sits_out_needs_no_state(first):
    """No kernel of a call touches a context with max_steps = 0, so it may be
    one without device state, particles or lists."""
    import torch
    say(f"batched device loop: a context without state sits out (first: {first})")
    stream = torch.cuda.Stream()
    alone, batched = (resident(1300, 94, stream) for _ in range(2))
    bare = B.Context(n_max=64, node_max=16, group_max=1, list_max=16, active_max=64, eps2=1e-4, precision="mixed",
                     stream=stream.cuda_stream)
    batch = batch_of(2, stream)
    order = [bare, batched.ctx] if first else [batched.ctx, bare]
    handles = np.array([c.handle.value for c in order], np.uint64)
    k, t, p = alone.ctx.dev_run(0.02, 1.0 / 64, 1.0 / 64, 25)
    steps, t_last, psteps, pairs, step_ms = batch.dev_run(handles, [0.02] * 2, [1.0 / 64] * 2, [1.0 / 64] * 2,
                                                          [0 if c is bare else 25 for c in order], 32)
    runs, sits = order.index(batched.ctx), order.index(bare)
    assert (steps[runs], t_last[runs], psteps[runs]) == (k, t, p) and len(step_ms) == k > 0
    assert (steps[sits], psteps[sits], pairs[sits]) == (0, 0, 0) and np.isnan(t_last[sits])
    for q, w in zip(batched.ctx.state_get(), alone.ctx.state_get()):
        assert np.array_equal(q, w)
    # nobody runs: no step, nothing touched
    steps, _, _, _, step_ms = batch.dev_run(handles, [0.02] * 2, [1.0 / 64] * 2, [1.0 / 64] * 2, [0, 0], 32)
    assert not steps.any() and len(step_ms) == 0
    for s in (alone, batched, bare, batch):
        s.close()
