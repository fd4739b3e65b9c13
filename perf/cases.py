"""The work that users of this framework have it do, as cases that can be timed and compared.

A case names one of six kinds of pass through the public entry points (paper_1602_02832_amd.binding):

  step      one block step of a host-driven integration: j-memory update, prediction and list force of the
            active particles in one call (Context.step_async)
  force     prediction and list force of an active set (Context.predict, Context.force_async): the
            all-particle step at a tree time, and the eager form of prediction
  direct    the direct N^2 sum over all particles (Context.force_direct_async)
  tree      keys, order, octree, node moments, groups and lists on the device (DeviceTree.build)
  interval  a resident cluster taken through block steps on the device (Context.state_set, dev_run, state_get)
  ensemble  several resident clusters stepped together (Batch.dev_run)

Inputs are Plummer models in standard units (G = M = -4E = 1), the accelerations and jerks of the mean field,
and block steps from Aarseth's first criterion with the scatter that encounters give.  The tree and lists that
a force pass needs in hand are made here in plain torch, from the definitions in include/htree_tree.h.
"""
import math

import numpy as np
import torch

from paper_1602_02832_amd import binding as B
from paper_1602_02832_amd.driver import Simulation

_SCALE = 3.0 * math.pi / 16.0   # Plummer length in standard units
_LEVELS = 21                    # bits per axis of the Peano-Hilbert key, and the deepest cell level


def listed():
    one_m = {"n": 1 << 20, "theta": 0.4, "n_crit": 2048, "dt_tree": 1.0 / 512, "precision": "mixed", "predict": "fused"}
    small = {"n": 16384, "theta": 0.4, "n_crit": 256, "dt_tree": 1.0 / 256, "precision": "fp64", "predict": "fused"}
    return [
        # the smallest call: one particle due in a cluster of two thousand, where only latency counts
        {"name": "step_2k_1", "kind": "step", "n": 2048, "theta": 0.5, "n_crit": 64, "dt_tree": 1.0 / 128,
         "precision": "fp64", "predict": "fused", "n_active": 1},
        # an ordinary step of a 16 thousand particle run in the FP64 form
        {"name": "step_16k_200", "kind": "step", "n_active": 197, **small},
        # the median, the mean and the largest ordinary step of the million-particle run
        {"name": "step_1m_27", "kind": "step", "n_active": 27, **one_m},
        {"name": "step_1m_559", "kind": "step", "n_active": 559, **one_m},
        {"name": "step_1m_6313", "kind": "step", "n_active": 6313, **one_m},
        # its all-particle step, taken at every tree time
        {"name": "all_1m", "kind": "force", "n_active": 1 << 20, **one_m},
        # the all-particle step of a middle-sized cluster, FP64 form, predicted eagerly
        {"name": "all_65k_eager", "kind": "force", "n_active": 65536, "n": 65536, "theta": 0.5, "n_crit": 256,
         "dt_tree": 1.0 / 256, "precision": "fp64", "predict": "eager"},
        # the direct scheme's mean step, which the tree is compared with
        {"name": "direct_1m_559", "kind": "direct", "n_active": 559, **one_m},
        # the rebuild at a tree time: the million-particle run, and a small odd-sized cluster
        {"name": "tree_1m", "kind": "tree", **one_m},
        {"name": "tree_20k", "kind": "tree", **{**small, "n": 20011}},
        # one cluster handed over, taken through 64 block steps on the device and handed back
        {"name": "interval_16k", "kind": "interval", "steps": 64, "eta": 0.01, **{**small, "precision": "mixed"}},
        # eight clusters of 4 to 64 thousand particles stepped together, as the batched engine does
        {"name": "ensemble_8", "kind": "ensemble", "clusters": 8, "n": 4096, "n_high": 65536, "theta": 0.5,
         "n_crit": 256, "dt_tree": 1.0 / 256, "precision": "mixed", "predict": "fused", "steps": 32, "eta": 0.01},
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "force", "direct", "tree", "interval", "ensemble"])
    n = _log_int(rng, 2048, 1 << 20)
    c = {"kind": kind, "n": n, "theta": rng.choice([0.3, 0.4, 0.5, 0.75]), "dt_tree": 1.0 / rng.choice([128, 256, 512]),
         "precision": rng.choice(["mixed", "mixed", "fp64"]), "predict": "fused"}
    lo = max(64, n // 2048)   # as the configurations do: some hundreds to thousands of groups
    c["n_crit"] = _log_int(rng, lo, max(lo + 1, min(2048, n // 16)))
    if kind == "step":
        c["n_active"] = _log_int(rng, 1, max(2, n // 64))
    elif kind == "force":
        # the largest all-particle pass stays below the listed one: theta 0.3's lists are twice as long
        c["n"], c["theta"] = min(n, 300000), max(c["theta"], 0.4)
        c["n_active"] = rng.choice([c["n"], _log_int(rng, c["n"] // 64, c["n"])])
        c["predict"] = rng.choice(["fused", "eager"])
    elif kind == "direct":
        c["n_active"] = _log_int(rng, 1, min(n, (1 << 29) // n))
    elif kind == "interval":
        c["n"] = _log_int(rng, 2048, 65536)
        c["n_crit"] = _log_int(rng, 64, 512)
        c["steps"], c["eta"] = _log_int(rng, 16, 64), 0.01
    elif kind == "ensemble":
        c["clusters"], c["n_high"] = rng.randint(3, 8), _log_int(rng, 8192, 65536)
        c["n"] = _log_int(rng, 1024, 8192)
        c["n_crit"] = _log_int(rng, 64, 512)
        c["theta"] = max(c["theta"], 0.4)
        c["steps"], c["eta"] = _log_int(rng, 8, 32), 0.01
    return c


# ------------------------------------------------------------------------------------------------- inputs
def _isotropic(r, gen):
    u = torch.rand((2, r.shape[0]), generator=gen, device=r.device, dtype=r.dtype)
    cos, phi = 2.0 * u[0] - 1.0, 2.0 * math.pi * u[1]
    sin = (1.0 - cos * cos).sqrt()
    return torch.stack([r * sin * phi.cos(), r * sin * phi.sin(), r * cos], 1)


def _plummer(n, seed):
    """x, v, m of a Plummer model (Aarseth, Henon & Wielen's sampling; enclosed mass cut at 0.999)."""
    gen = torch.Generator("cuda").manual_seed(seed)
    f64 = {"device": "cuda", "dtype": torch.float64}
    r = ((torch.rand(n, generator=gen, **f64) * 0.999).clamp_min(1e-12) ** (-2.0 / 3.0) - 1.0).rsqrt()
    x = _isotropic(r, gen)
    q = torch.zeros(n, **f64)
    todo = torch.arange(n, device="cuda")
    while todo.numel():
        u = torch.rand((2, todo.numel()), generator=gen, **f64)
        ok = 0.1 * u[1] < u[0] ** 2 * (1.0 - u[0] ** 2) ** 3.5
        q[todo[ok]] = u[0][ok]
        todo = todo[~ok]
    v = _isotropic(q * math.sqrt(2.0) * (1.0 + r * r) ** -0.25, gen)
    # masses: Salpeter's spectrum over a factor of a hundred, total 1
    p = 1.0 - 2.35
    m = (1.0 + torch.rand(n, generator=gen, **f64) * (100.0 ** p - 1.0)) ** (1.0 / p)
    return x * _SCALE, v / math.sqrt(_SCALE), m / m.sum()


def _spread(c):
    """Bit k of c to bit 3 k."""
    for s, mask in ((32, 0x1F00000000FFFF), (16, 0x1F0000FF0000FF), (8, 0x100F00F00F00F00F), (4, 0x10C30C30C30C30C3),
                    (2, 0x1249249249249249)):
        c = (c | (c << s)) & mask
    return c


def _hilbert(x):
    """63-bit Peano-Hilbert keys (Skilling 2004) in the power-of-two cube at the componentwise minimum; its side."""
    lo = x.amin(0)
    ext = float((x.amax(0) - lo).max())
    side = math.ldexp(1.0, math.frexp(ext)[1]) if ext > 0 else 1.0
    c = list(((x - lo) * (2.0 ** _LEVELS / side)).floor().clamp(0, 2 ** _LEVELS - 1).to(torch.int64).unbind(1))
    for b in range(_LEVELS - 1, 0, -1):
        for d in range(3):
            on = ((c[d] >> b) & 1).bool()
            swap = torch.where(on, 0, (c[0] ^ c[d]) & ((1 << b) - 1))
            c[0] = torch.where(on, c[0] ^ ((1 << b) - 1), c[0] ^ swap)
            c[d] = c[d] ^ swap if d else c[0]
    c[1] = c[1] ^ c[0]
    c[2] = c[2] ^ c[1]
    flip = torch.zeros_like(c[0])
    for b in range(_LEVELS - 1, 0, -1):
        flip ^= ((c[2] >> b) & 1) * ((1 << b) - 1)
    return (_spread(c[0] ^ flip) << 2) | (_spread(c[1] ^ flip) << 1) | _spread(c[2] ^ flip), side


def _tree(x, v, a, j, m, n_crit, theta):
    """The octree over particles (leaves of one), its node moments, groups and lists.  Everything in key order;
    list entries and cells are combined indices (particle k is k, node q is n + q)."""
    n = x.shape[0]
    keys, side = _hilbert(x)
    keys, perm = torch.sort(keys, stable=True)
    x, v, a, j, m = (u[perm].contiguous() for u in (x, v, a, j, m))
    begin, end, level = [], [], []
    for lv in range(_LEVELS + 1):   # a node is a cell of at least two particles
        _, count = torch.unique_consecutive(keys >> (3 * (_LEVELS - lv)), return_counts=True)
        stop = count.cumsum(0)
        many = count > 1
        begin.append((stop - count)[many])
        end.append(stop[many])
        level.append(torch.full_like(begin[-1], lv))
    begin, end, level = torch.cat(begin), torch.cat(end), torch.cat(level)
    order = torch.argsort(begin * 32 + level)
    begin, end, level = begin[order], end[order], level[order]
    # parents: the node one level up for a node, the deepest node around it for a particle
    particle = torch.arange(n, device=x.device)
    parent = torch.full((n + begin.shape[0],), -1, device=x.device)
    ids = torch.arange(begin.shape[0], device=x.device)
    for lv in range(int(level.max()) + 1):
        here = level == lv
        b, e, q = begin[here], end[here], ids[here]
        if lv < int(level.max()):
            below = level == lv + 1
            parent[n + ids[below]] = q[torch.searchsorted(b, begin[below], right=True) - 1]
        at = (torch.searchsorted(b, particle, right=True) - 1).clamp_min(0)
        parent[:n] = torch.where((b[at] <= particle) & (particle < e[at]), q[at], parent[:n])
    cell_begin, cell_end = torch.cat([particle, begin]), torch.cat([particle + 1, end])
    rank = torch.cat([particle * 32 + 31, begin * 32 + level])   # pre-order
    kids = torch.argsort(parent * n + cell_begin, stable=True)[1:]   # by parent, in key order, without the root
    n_kids = torch.bincount(parent[kids], minlength=begin.shape[0])
    first_kid = n_kids.cumsum(0) - n_kids
    # moments, from the deepest level up
    sums = torch.zeros((n + begin.shape[0], 13), device=x.device, dtype=x.dtype)
    sums[:n] = m[:, None] * torch.cat([torch.ones_like(m)[:, None], x, v, a, j], 1)
    for lv in range(int(level.max()), -1, -1):
        q = ids[level == lv]
        rows = kids[_ranges(first_kid[q], n_kids[q])]
        sums[n + q] = torch.segment_reduce(sums[rows], "sum", lengths=n_kids[q], axis=0, unsafe=True)
    node_m = sums[n:, 0].contiguous()
    mean = sums[n:, 1:] / node_m[:, None]
    # groups: the first cells from the root with at most n_crit particles
    size = cell_end - cell_begin
    above = torch.where(parent >= 0, size[n + parent.clamp_min(0)], n_crit + 1)
    group = torch.sort(cell_begin[(size <= n_crit) & (above > n_crit)])[0]
    group_first = torch.cat([group, group.new_tensor([n])])
    of = (torch.searchsorted(group, particle, right=True) - 1)[:, None].expand(n, 3)
    lo = x.new_full((group.shape[0], 3), math.inf).scatter_reduce(0, of, x, "amin")
    hi = x.new_full((group.shape[0], 3), -math.inf).scatter_reduce(0, of, x, "amax")
    side2 = torch.tensor([(side * 0.5 ** k) ** 2 for k in range(_LEVELS + 1)], device=x.device, dtype=x.dtype)
    # lists: all groups go down the tree together, a level at a time
    found = []
    g, c = torch.arange(group.shape[0], device=x.device), torch.full_like(group, n)
    while g.numel():
        leaf = c < n
        q = (c - n).clamp_min(0)
        gap = torch.maximum(lo[g] - mean[q, :3], mean[q, :3] - hi[g]).clamp_min(0.0)
        far = side2[level[q]] < theta * theta * (gap * gap).sum(1)
        apart = (cell_end[c] <= group_first[g]) | (group_first[g + 1] <= cell_begin[c])
        done = leaf | (far & apart)
        found.append(torch.stack([g[done], c[done]]))
        g, q = g[~done], q[~done]
        g, c = g.repeat_interleave(n_kids[q]), kids[_ranges(first_kid[q], n_kids[q])]
    g, c = torch.cat(found, 1)
    at = torch.argsort(g * (32 * n) + rank[c])
    list_off = torch.zeros(group.shape[0] + 1, dtype=torch.int64, device=x.device)
    list_off[1:] = torch.bincount(g, minlength=group.shape[0]).cumsum(0)
    return {"perm": perm, "keys": keys, "x": x, "v": v, "a": a, "j": j, "m": m, "node_m": node_m,
            "node_x": mean[:, 0:3].contiguous(), "node_v": mean[:, 3:6].contiguous(),
            "node_a": mean[:, 6:9].contiguous(), "node_j": mean[:, 9:12].contiguous(), "group_first": group_first,
            "list_off": list_off, "entries": c[at].to(torch.int32)}


def _ranges(first, count):
    """first[0], first[0] + 1, ... (count[0] of them), first[1], ..."""
    stop = count.cumsum(0)
    total = int(stop[-1]) if count.numel() else 0
    return torch.arange(total, device=first.device) + (first - stop + count).repeat_interleave(count)


def _particles(case, seed):
    """Particles with the mean field's acceleration and jerk, in any order.  A tree pass gets the same places for
    every seed, so that its results have the same sizes, in another order and with other velocities."""
    x, v, m = _plummer(case["n"], seed)
    if case["kind"] == "tree":
        gen = torch.Generator("cuda").manual_seed(seed + 1)
        order = torch.randperm(case["n"], generator=gen, device="cuda")
        x, _, m = (u[order] for u in _plummer(case["n"], 11))
    s = (x * x).sum(1, keepdim=True) + _SCALE * _SCALE
    a = -x * s ** -1.5
    j = -v * s ** -1.5 + 3.0 * (x * v).sum(1, keepdim=True) * x * s ** -2.5
    return x, v, a, j, m


def _eps2(n):
    return (4.0 / n) ** 2


def _scene(case, seed):
    """Tree, lists and block state at a block time: t, every particle's t0 < t, and the active ids."""
    x, v, a, j, m = _particles(case, seed)
    s = _tree(x, v, a, j, m, case["n_crit"], case["theta"])
    n, top = case["n"], case["dt_tree"]
    gen = torch.Generator("cuda").manual_seed(seed + 1)
    scatter = torch.randn(n, generator=gen, device="cuda", dtype=torch.float64)
    raw = 0.01 * s["a"].norm(dim=1) / s["j"].norm(dim=1) * torch.exp(scatter - 2.0)
    dt = (2.0 ** raw.log2().floor()).clamp(top * 2.0 ** -12, top)
    s["t"] = top * 0.8125
    s["t0"] = ((s["t"] / dt).ceil() - 1.0) * dt
    s["active"] = torch.sort(torch.argsort(raw, stable=True)[:case["n_active"]])[0].to(torch.int32)
    return s


def _context(case, s, stream):
    n = case["n"]
    c = B.Context(n_max=n, node_max=s["node_m"].shape[0], group_max=s["group_first"].shape[0] - 1,
                  list_max=s["entries"].shape[0], active_max=n, eps2=_eps2(n), precision=case["precision"],
                  predict_mode=case["predict"], stream=stream)
    h = {k: s[k].cpu().numpy() for k in ("t0", "m", "x", "v", "a", "j", "node_m", "node_x", "node_v", "node_a",
                                         "node_j", "group_first", "list_off", "entries")}
    c.set_j_particles(h["t0"], h["m"], h["x"], h["v"], h["a"], h["j"])
    c.set_nodes(0.0, h["node_m"], h["node_x"], h["node_v"], h["node_a"], h["node_j"])
    c.set_interaction_lists(h["group_first"], h["list_off"], h["entries"])
    return c


def _simulation(case, n, seed, stream):
    """A resident cluster at t = 0 with its first forces and block steps, and a host copy of its state."""
    x, v, m = (u.cpu().numpy() for u in _plummer(n, seed))
    sim = Simulation(x, v, m, eps2=_eps2(n), dt_tree=case["dt_tree"], eta=case["eta"], theta=case["theta"],
                     n_crit=case["n_crit"], precision=case["precision"], resident=True, device_loop=True, stream=stream)
    t0, dt, x, v, a, j, pot = sim.ctx.state_get()
    return sim, (t0, dt, sim.m, x, v, a, j, pot)


def _ensemble_sizes(case):
    lo, hi, k = math.log(case["n"]), math.log(case["n_high"]), case["clusters"]
    return [int(math.exp(lo + (hi - lo) * (i + 0.5) / k)) for i in range(k)]


def prepare(case, seed):
    kind = case["kind"]
    stream = torch.cuda.Stream()
    if kind == "tree":
        part = [u.contiguous() for u in _particles(case, seed)]
        torch.cuda.synchronize()
        return {"case": case, "part": part, "tree": B.DeviceTree(n_max=case["n"]), "views": {}}
    if kind == "interval":
        sim, state = _simulation(case, case["n"], seed, stream.cuda_stream)
        return {"case": case, "stream": stream, "sim": sim, "state": state}
    if kind == "ensemble":
        made = [_simulation(case, n, seed + 100 * k, stream.cuda_stream) for k, n in enumerate(_ensemble_sizes(case))]
        sims = [sim for sim, _ in made]
        total = sum(sim.n for sim in sims)
        batch = B.Batch(stream=stream.cuda_stream, max_clusters=len(sims), max_items=16 * total, max_active=total,
                        max_rows=total)
        return {"case": case, "stream": stream, "sims": sims, "states": [state for _, state in made], "batch": batch,
                "handles": np.array([sim.ctx.handle.value for sim in sims], np.uint64)}
    s = _scene(case, seed)
    ctx = _context(case, s, stream.cuda_stream)
    k = case["n_active"]
    out = {name: torch.zeros((k, 3) if name != "pot" else k, device="cuda", dtype=torch.float64)
           for name in ("acc", "jerk", "pot")}
    st = {"case": case, "stream": stream, "ctx": ctx, "t": s["t"], "active": s["active"].cpu().numpy(), "out": out,
          "to": tuple(u.data_ptr() for u in out.values())}
    if kind == "step":   # the rows that the last step's corrector left on the device
        ids = s["active"].long()
        rows = [s["active"].contiguous()] + [s[f][ids].contiguous() for f in ("t0", "m", "x", "v", "a", "j")]
        st["rows"], st["update"] = rows, (k, *(u.data_ptr() for u in rows))
        st["ids"] = (k, st["active"].ctypes.data)
    torch.cuda.synchronize()
    return st


class _View:
    """Device memory of the library's as an array that torch can take; a tensor of it keeps `owner` alive."""

    def __init__(self, owner, address, shape, kind):
        self.owner = owner
        self.__cuda_array_interface__ = {"data": (address, False), "shape": shape, "typestr": kind, "version": 2}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        state["ctx"].step_async(state["update"], state["t"], state["ids"], *state["to"])
        return state["out"]
    if kind in ("force", "direct"):
        ctx, out = state["ctx"], state["out"]
        ctx.predict(state["t"])
        force = ctx.force_async if kind == "force" else ctx.force_direct_async
        force(state["active"], out["acc"], out["jerk"], out["pot"])
        return out
    if kind == "tree":
        tree = state["tree"]
        nodes, groups, entries, _ = tree.build(*state["part"], 1, case["n_crit"], case["theta"])
        view, n = tree.view(), case["n"]
        out = {}
        for name, shape, typ in (("perm", (n,), "<i8"), ("keys", (n,), "<i8"), ("node_m", (nodes,), "<f8"),
                                 ("node_x", (nodes, 3), "<f8"), ("node_v", (nodes, 3), "<f8"),
                                 ("node_a", (nodes, 3), "<f8"), ("node_j", (nodes, 3), "<f8"),
                                 ("group_first", (groups + 1,), "<i8"), ("list_off", (groups + 1,), "<i8"),
                                 ("entries", (entries,), "<i4")):
            at = (getattr(view, name), shape)
            held = state["views"].get(name)
            if held is None or held[0] != at:   # the tensors follow the tree's arrays when these move or grow
                held = state["views"][name] = (at, torch.as_tensor(_View(tree, *at, typ), device="cuda"))
            out[name] = held[1]
        return out
    if kind == "interval":
        ctx = state["sim"].ctx
        ctx.state_set(*state["state"])
        steps, t_last, psteps = ctx.dev_run(case["eta"], case["dt_tree"], case["dt_tree"], case["steps"])
        return {"steps": steps, "t_last": t_last, "particle_steps": psteps, "state": ctx.state_get()}
    sims, k = state["sims"], len(state["sims"])
    for sim, s in zip(sims, state["states"]):
        sim.ctx.state_set(*s)
    tops = np.full(k, case["dt_tree"])
    done = state["batch"].dev_run(state["handles"], np.full(k, case["eta"]), tops, tops,
                                  np.full(k, case["steps"], np.int32), case["steps"])
    return {"steps": done[0], "t_last": done[1], "particle_steps": done[2], "pairs": done[3],
            "states": [sim.ctx.state_get() for sim in sims]}


# ------------------------------------------------------------------------------------------------- measures
def _list_pairs(s):
    """(pairs, distinct entries, list indices) of the active particles' groups."""
    group = torch.searchsorted(s["group_first"], s["active"].long(), right=True) - 1
    g, count = torch.unique_consecutive(group, return_counts=True)
    length = s["list_off"][g + 1] - s["list_off"][g]
    used = torch.zeros(s["m"].shape[0] + s["node_m"].shape[0], dtype=torch.bool, device="cuda")
    used[s["entries"][_ranges(s["list_off"][g], length)].long()] = True
    return int((count * length).sum()), int(used.sum()), int(length.sum())


def work(case):
    """57 operations a pair (the paper's count); every record (84 bytes in the mixed form, 112 in FP64), list index
    and active id read once, every result written once."""
    kind, n = case["kind"], case["n"]
    rec = 84 if case["precision"] == "mixed" else 112
    if kind in ("step", "force"):
        pairs, used, index = _list_pairs(_scene(case, 1))
        moved = used * rec + index * 4 + case["n_active"] * 60
        if kind == "step":
            moved += case["n_active"] * (116 + rec)
        return {"bytes": moved, "flops": 57.0 * pairs}
    if kind == "direct":
        return {"bytes": n * rec + case["n_active"] * 60, "flops": 57.0 * n * case["n_active"]}
    if kind == "tree":
        s = _tree(*_particles(case, 1), case["n_crit"], case["theta"])
        return {"bytes": n * (104 + 16 + 104) + s["node_m"].shape[0] * 104 + s["entries"].shape[0] * 4, "flops": 0}
    # a state handed over and back, and at each step the due times and about one list a step for a few particles
    sizes = [n] if kind == "interval" else _ensemble_sizes(case)
    total = sum(sizes)
    return {"bytes": total * (136 + 128) + case["steps"] * total * 16, "flops": 57.0 * case["steps"] * 16 * 2000 * len(sizes)}


def _pair_sums(xi, vi, xj, vj, mj, eps2, same):
    """a, jerk and potential of the particles i from the entries j; same: pairs of a particle with itself."""
    dx, dy, dz = (xj[None, :, d] - xi[:, None, d] for d in range(3))
    wx, wy, wz = (vj[None, :, d] - vi[:, None, d] for d in range(3))
    inv = (dx * dx + dy * dy + dz * dz + eps2).rsqrt().masked_fill_(same, 0.0)
    mr = mj * inv
    inv = inv * inv
    c = (dx * wx + dy * wy + dz * wz).mul_(inv).mul_(3.0)
    mr3 = mr * inv
    acc = torch.stack([(mr3 * d).sum(1) for d in (dx, dy, dz)], 1)
    jerk = torch.stack([(mr3 * (w - c * d)).sum(1) for d, w in ((dx, wx), (dy, wy), (dz, wz))], 1)
    return acc, jerk, -mr.sum(1)


def exact(case, seed):
    """The same sums in 64 bits, from the unrounded inputs.  None for whole integrations, whose block steps follow
    from every force before them."""
    kind = case["kind"]
    if kind in ("interval", "ensemble"):
        return None
    if kind == "tree":
        s = _tree(*_particles(case, seed), case["n_crit"], case["theta"])
        floats = ("node_m", "node_x", "node_v", "node_a", "node_j")
        return {k: s[k] if k in floats else None for k in ("perm", "keys", *floats, "group_first", "list_off", "entries")}
    s = _scene(case, seed)
    n = case["n"]

    def predicted(h, x, v, a, j):
        return x + h * (v + h / 2.0 * (a + h / 3.0 * j)), v + h * (a + h / 2.0 * j)

    xp, vp = predicted((s["t"] - s["t0"])[:, None], s["x"], s["v"], s["a"], s["j"])
    nx, nv = predicted(s["t"], s["node_x"], s["node_v"], s["node_a"], s["node_j"])
    x, v, m = torch.cat([xp, nx]), torch.cat([vp, nv]), torch.cat([s["m"], s["node_m"]])
    active = s["active"].long()
    if kind == "direct":
        parts = [(i, torch.arange(n, device="cuda")) for i in active.split(max(1, 40_000_000 // n))]
    else:
        group = torch.searchsorted(s["group_first"], active, right=True) - 1
        g, count = torch.unique_consecutive(group, return_counts=True)
        off = s["list_off"].tolist()
        parts = []
        for q, i in zip(g.tolist(), active.split(count.tolist())):
            e = s["entries"][off[q]:off[q + 1]].long()
            parts += [(k, e) for k in i.split(max(1, 40_000_000 // max(1, e.numel())))]
    got = [_pair_sums(x[i], v[i], x[e], v[e], m[e], _eps2(n), i[:, None] == e[None, :]) for i, e in parts]
    return dict(zip(("acc", "jerk", "pot"), (torch.cat(u) for u in zip(*got))))
