"""The ways in which the parts of split walks are kept and added, each on a
cloud that takes it:

* clouds that fill the chip: FP32 parts, few or many per group, added by the
  moment pass that follows (few or many loads in flight);
* smaller ones: FP64 parts, few per group, added by the moment pass;
* walks planned beyond 4,096 visits, cut at two split sizes that differ.

Combining inside the moment pass is the separate launch's arithmetic in its
order: identical bit for bit.  Split walks make the decisions of whole walks:
equal pair counts, sums within `parity_bar.same_terms`.
"""
import numpy as np
import pytest

import parity_bar
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16634_amd as w
    w.load_library()
    return torch.device("cuda:0")


# points, split, parts per group: at least, at most
PATHS = {"fp32_few": (400000, 256, 2, 8), "fp32_many": (400000, 64, 9, 40),
         "fp64_few": (150000, 256, 4, 8)}


@pytest.mark.parametrize("path", list(PATHS))
def test_combining_in_the_moment_pass_is_bit_identical(dev, path):
    import torch
    import paper_2405_16634_amd as w
    n, split, lo, hi = PATHS[path]
    print(f"[case] part paths {path}", flush=True)
    ctx = w.Context(0)
    x, _ = ctx.normalize(torch.from_numpy(synth.torus_knot(n, 5, with_init=False).points).to(dev))
    ctx.build(x)
    ctx.set_split(split)
    st = ctx.stats()
    per = st["n_tasks"] / st["n_groups"]
    print(f"  {per:.1f} parts per group", flush=True)
    assert lo <= per <= hi
    res = []
    for flags in (0, w.FLAG_SEPARATE_COMBINE):
        ctx.set_flags(flags)
        mu = ctx.orient(3, 0.002, 0.016).clone()
        e = np.asarray(ctx.energy(3)).copy()
        ctx.set_flags(flags | w.FLAG_TIME_KERNELS)
        ctx.reset_stats()
        ctx.orient(3, 0.002, 0.016)
        res.append((mu, e, ctx.stats()["combine_ms"]))
        ctx.set_flags(0)
    assert bool((res[0][0] == res[1][0]).all()) and np.array_equal(res[0][1], res[1][1])
    assert bool(torch.isfinite(res[0][0]).all())
    # the separate launches' time: of 11 walks in 3 iterations, or of the 4
    # that no moment pass follows
    assert 0 < res[0][2] < 0.7 * res[1][2]
    ctx.close()


def test_long_planned_walks_cut_at_two_sizes(dev, oracle_mod):
    import torch
    import paper_2405_16634_amd as w
    n, c = 12000, 8.0
    print("[case] part paths long walks", flush=True)
    rng = np.random.default_rng(6)
    ctx = w.Context(0)
    x, _ = ctx.normalize(torch.from_numpy(synth.torus_knot(n, 5, with_init=False).points).to(dev))
    ctx.build(x, c)
    mu = (synth.random_unit(rng, n) * 1e-3).astype(np.float32)
    rho = rng.standard_normal(n).astype(np.float32)
    mu_d, rho_d = torch.from_numpy(mu).to(dev), torch.from_numpy(rho).to(dev)
    res, tasks = {}, {}
    for split in (0, 24, 1024):
        ctx.set_split(split)
        ctx.set_flags(w.FLAG_COUNT_PAIRS)
        ctx.reset_stats()
        out = [ctx.winding(mu_d, 0.002).cpu().numpy(), ctx.gradient(mu_d, 0.002).cpu().numpy(),
               ctx.adjoint(rho_d, 0.002).cpu().numpy()]
        st = ctx.stats()
        ctx.set_flags(0)
        res[split], tasks[split] = (out, list(st["pairs"])), st["n_tasks"]
    ctx.close()
    print(f"  tasks {tasks}", flush=True)
    assert tasks[24] > 1.2 * tasks[1024] > 10 * tasks[0]
    T = oracle_mod.Tree(x.cpu().numpy().astype(np.float64))
    for q, (op, nu) in enumerate((("A", mu), ("G", mu), ("AT", rho))):
        mag = T.apply(op, nu.astype(np.float64), 0.002, c, with_stats=True)[1]
        for split in (24, 1024):
            assert res[split][1] == res[0][1], split
            parity_bar.same_terms(f"split={split} {op}", res[split][0][q], res[0][0][q], mag)


def test_long_planned_walks_of_a_wide_tree(dev):
    """Exact sums of a tree of more than 2^16 nodes (child offsets beyond 16
    bits): split walks count the pairs of whole walks, and every target's sum
    of n terms agrees to 1e-6 of the largest."""
    import torch
    import paper_2405_16634_amd as w
    n = 60000
    print("[case] part paths wide", flush=True)
    ctx = w.Context(0)
    x, _ = ctx.normalize(torch.from_numpy(synth.fibonacci_sphere(n, 1).points).to(dev))
    ctx.build(x, 1e6)
    assert ctx.stats()["n_nodes"] > 1 << 16
    mu = torch.from_numpy((synth.random_unit(np.random.default_rng(2), n) * 1e-3).astype(np.float32)).to(dev)
    ctx.set_flags(w.FLAG_COUNT_PAIRS)
    out, pairs = [], []
    for split in (0, 256):
        ctx.set_split(split)
        ctx.reset_stats()
        out.append(ctx.gradient(mu, 0.002).double())
        pairs.append(ctx.stats()["pairs"][2])
    ctx.close()
    assert pairs[0] == pairs[1] == n * n
    assert float((out[0] - out[1]).abs().max()) <= 1e-6 * float(out[0].abs().max())
