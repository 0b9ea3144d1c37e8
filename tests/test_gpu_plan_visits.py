"""The parts of split walks against the walks themselves.

The nodes that a 64-target group's walk visits are counted here in numpy from
the exported tree and the representatives of a constant attribute (the
attribute that walks are planned with), in FP32 as on the device.  From the
visits V of every group follows the number of tasks: parts of

    visits per part = the split size, or less on clouds whose walks are fewer
                      parts of that size than fill the chip: as many visits as
                      make 8,192 parts, if that is 120 or less, else 16,384

that is ceil(V / that) parts per group, cut at the plan's nodes.  A distance on
the threshold may fall either way, so the counts may differ by 1 %.

Walks of more than 4,096 visits (a large c) are planned by a kernel of their
own.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
FILL = 16384


def walk_visits(ctx, x, c, group=64):
    """Visits of every group's walk (one cloud)."""
    import torch
    if c >= 1e5:  # every node
        return np.full(-(-len(x) // group), ctx.stats()["n_nodes"])
    depth, leaf, begin, end, perm = ctx.tree()
    xB = ctx.moments(torch.full((len(x),), 0.5, device=x.device))[0]
    m = len(depth)
    parent = np.full(m, -1)
    last = {}
    for k, d in enumerate(depth.tolist()):
        last[d] = k
        if d > 0:
            parent[k] = last[d - 1]
    order = np.argsort(parent[1:], kind="stable") + 1  # children by parent
    first = np.searchsorted(parent[order], np.arange(m + 1))
    thr2 = (np.float32(c) * np.ldexp(np.float32(1), 1 - depth).astype(np.float32)) ** 2
    inner = leaf == 0
    X = x.cpu().numpy()[perm]
    V = []
    for a in range(0, len(X), group):
        t = X[a:a + group]
        nodes, total = np.array([0]), 1
        while len(nodes):
            nodes = nodes[inner[nodes]]
            d2 = np.full(len(nodes), np.inf, np.float32)
            for p in t:
                d2 = np.minimum(d2, ((p - xB[nodes]) ** 2).sum(1))
            nodes = nodes[d2 <= thr2[nodes]]
            nodes = np.concatenate([order[first[k]:first[k + 1]] for k in nodes]) if len(nodes) else nodes
            total += len(nodes)
        V.append(total)
    return np.array(V)


def expected_tasks(V, split):
    """ceil(V / visits per part) per group, cut at one of up to 256 nodes."""
    fill, one = int(V.sum()) // FILL, int(V.sum()) // (FILL // 2 - len(V) // 2) + 1
    per = min(split, max(one if one <= 120 else fill, 16))
    step = np.full(len(V), 16)
    while (256 * step < V).any():
        step[256 * step < V] *= 2
    return int(np.minimum(np.ceil(V / per), (V - 1) // step + 1).sum())


@pytest.mark.parametrize("n,c", [(4000, 6.0), (20000, 8.0), (9000, 1e6), (20000, 1e6), (60000, 1e6)])
def test_long_walks_are_cut_evenly(n, c):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16634_amd as w
    w.load_library()
    print(f"[case] plan visits {n} c={c}", flush=True)
    dev = torch.device("cuda:0")
    ctx = w.Context(0)
    x, _ = ctx.normalize(torch.from_numpy(synth.torus_knot(n, 5, with_init=False).points).to(dev))
    ctx.build(x, c)
    V = walk_visits(ctx, x, c)
    got = ctx.stats()["n_tasks"]
    print(f"  visits {V.min()}..{V.max()}, tasks {got}, expected {expected_tasks(V, 256)}", flush=True)
    if n > 4000:
        assert V.max() > 4096
    assert abs(got - expected_tasks(V, 256)) <= 0.01 * got
    ctx.close()


@pytest.mark.parametrize("n,c", [(2000, 2.0), (30000, 2.0), (20000, 8.0)])
def test_smaller_splits_never_make_longer_parts(n, c):
    """Clouds that parts of 64 visits do not fill (2,000 and 30,000 points) and
    do fill (c = 8)."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16634_amd as w
    w.load_library()
    print(f"[case] splits {n} c={c}", flush=True)
    ctx = w.Context(0)
    x, _ = ctx.normalize(torch.from_numpy(synth.fibonacci_sphere(n, 1).points).to("cuda:0"))
    ctx.build(x, c)
    tasks = []
    for split in (0, 4096, 256, 128, 64, 63, 48, 33, 32, 17, 16, 1):
        ctx.set_split(split)
        st = ctx.stats()
        tasks.append(st["n_tasks"])
        if split == 0:
            assert st["n_tasks"] == st["n_groups"]
    print(f"  tasks {tasks}", flush=True)
    assert all(a <= b for a, b in zip(tasks, tasks[1:])), tasks
    assert tasks[1] >= 4 * tasks[0]
    ctx.close()


def test_forests_that_fill_the_chip_keep_most_walks_whole():
    """6,144 groups of walks that are on average shorter than the split size;
    a third of as many groups are cut into shorter parts."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16634_amd as w
    w.load_library()
    rng = np.random.default_rng(4)
    for clouds, whole in ((3072, True), (1024, False)):
        print(f"[case] forest of {clouds}", flush=True)
        p = torch.from_numpy(synth.random_unit(rng, 128 * clouds).astype(np.float32)).to("cuda:0")
        off = [128 * k for k in range(clouds + 1)]
        ctx = w.Context(0)
        x, _ = ctx.normalize_batched(p, off)
        ctx.build_batched(x, off)
        st = ctx.stats()
        ctx.close()
        assert st["n_groups"] == 2 * clouds
        if whole:
            assert st["n_tasks"] <= 1.05 * st["n_groups"], st
        else:
            assert st["n_tasks"] >= 3 * st["n_groups"], st
