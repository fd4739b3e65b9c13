"""Who sums the partials of split tiles: the tile's last item, or a launch after
the force, which sums up to 64 splits of a value in a thread and more through
LDS.  Direct sums against the oracle around those numbers of splits; batched
calls, whose contexts decide together, bit for bit against each context's own.
"""
import numpy as np
import pytest

from paper_1602_02832_amd import binding as B
from paper_1602_02832_amd import workloads as W

from parity_util import assert_close, say

pytestmark = pytest.mark.gpu


# a split of 256 entries each, and more than 16384 partial slots
@pytest.mark.parametrize("splits,k", [(8, 2049), (9, 1900), (16, 1030), (17, 1000), (64, 257), (64, 300), (65, 257), (66, 300)])
def test_many_splits_summed_by_a_launch(oracle, splits, k):
    n = 256 * (splits - 1) + 7 if k < 256 * (splits - 1) else 256 * splits + 7   # the last split is nearly empty
    splits = (n + 255) // 256
    say(f"direct sum: n={n} splits={splits} n_active={k}")
    assert k <= n and splits * k > 16384
    x, v, _ = W.plummer(n, 64)
    m = W.salpeter_masses(n, 65)
    z = np.zeros((n, 3))
    c = B.Context(n_max=n, node_max=16, group_max=1, list_max=16, active_max=n, eps2=1e-4, precision="fp64")
    c.set_j_particles(0.25, m, x, v, z, z)
    c.set_nodes(0.0, np.zeros(0), z[:0], z[:0], z[:0], z[:0])
    c.set_tuning(12, 1 << 20)
    c.predict(0.25)
    ids = np.sort(np.random.default_rng(k).choice(n, k, replace=False)).astype(np.int32)
    assert_close(f"splits {splits}", "fp64", c.force_direct(ids), oracle.force_direct(ids, x, v, m, 1e-4))
    c.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("count,k,target,most", [(2, 40, 1 << 20, 3072), (32, 60, 1 << 20, 0), (5, 2500, 1 << 20, 0),
                                                 (12, 1, 64, 3072)])
def test_batch_sums_equal_each_context_alone(oracle, prec, count, k, target, most):
    """Up to 3072 items of split tiles in a batch (most) and beyond."""
    import torch
    say(f"batched split sums: {count} contexts, {k} active, target {target}")
    n, t = 2500, 0.25
    stream = torch.cuda.Stream()
    ctxs, acts, outs = [], [], []
    for q in range(count):
        x, v, m = W.plummer(n, 300 + q)
        z = np.zeros((n, 3))
        tr = oracle.Tree(x, v, z, z, m, 1, 12, 0.3)
        x, v, m = x[tr.perm], v[tr.perm], m[tr.perm]
        c = B.Context(n_max=n, node_max=2 * n, group_max=n, list_max=2 * tr.n_entries, active_max=n, eps2=1e-4,
                      precision=prec, stream=stream.cuda_stream)
        c.set_j_particles(np.zeros(n), m, x, v, z, z)
        c.set_nodes(0.0, tr.node_m, tr.node_x, tr.node_v, tr.node_a, tr.node_j)
        c.set_interaction_lists(tr.group_first, tr.list_off, tr.entries)
        c.set_tuning(12, target)
        c.predict(t)
        ctxs.append(c)
        acts.append(np.sort(np.random.default_rng(q).choice(n, k, replace=False)).astype(np.int32))
        outs.append(tuple(torch.full(s, float("nan"), dtype=torch.float64, device="cuda") for s in ((k, 3), (k, 3), (k,))))
    batch = B.Batch(stream=stream.cuda_stream, max_clusters=count, max_items=1 << 17, max_active=count * n,
                    max_rows=count * n)
    torch.cuda.synchronize()
    batch.force_async(ctxs, acts, *zip(*outs))
    batch.sync()
    items = batch.last_stats()[1]
    assert (items <= most) if most else items > 3072, items
    for c, a, o in zip(ctxs, acts, outs):
        for got, want in zip(o, c.force(a)):
            assert np.array_equal(got.cpu().numpy(), want)
    for c in (*ctxs, batch):
        c.close()
