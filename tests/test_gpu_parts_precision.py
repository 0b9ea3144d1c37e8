"""Sums of split walks of small clouds: no less precise than whole walks.

The cloud is built with a huge c, so that every target opens every node and
its sum is the sum of the pair terms with the single points.  Only points no
two of which share a parent node have a non-zero attribute: the FP32 running
sums over siblings then hold at most one term each and are exact, and a walk's
result is the FP64 sum of its FP32 terms, rounded once at the end.  Parts of a
walk that keep FP64 sums give the same value up to

* the order of n FP64 additions, n 2^-53 of the term magnitudes M, and
* the final rounding of two such sums to FP32, 2^-23 of the value,

while parts rounded to FP32 miss it by about 2^-24 of the parts' magnitudes,
which the signs of the attributes make much larger than the value.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _support(tree, n, rng):
    """One point (caller row) below every node whose children hold a leaf."""
    depth, leaf, begin, end, perm = tree
    parent = np.full(len(depth), -1)
    last = {}
    for k, d in enumerate(depth):
        last[int(d)] = k
        if d > 0:
            parent[k] = last[int(d) - 1]
    assert np.all((end - begin)[leaf == 1] == 1)
    sel = {}
    for k in np.where(leaf == 1)[0]:
        sel.setdefault(int(parent[k]), int(begin[k]))
    return perm[np.array(sorted(sel.values()))]


@pytest.mark.parametrize("n", [150, 700, 1500])
def test_short_parts_keep_fp64_sums(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16634_amd as w
    w.load_library()
    print(f"[case] parts precision {n}", flush=True)
    rng = np.random.default_rng(11)
    dev = torch.device("cuda:0")
    ctx = w.Context(0)
    x, _ = ctx.normalize(torch.from_numpy(synth.fibonacci_sphere(n, 1).points).to(dev))
    ctx.build(x, 1e6)
    ctx.set_defer(0)
    rows = _support(ctx.tree(), n, rng)
    s = np.zeros(n, np.float32)
    s[rows] = rng.standard_normal(len(rows))
    mu = np.zeros((n, 3), np.float32)
    mu[rows] = rng.standard_normal((len(rows), 3))
    s_d, mu_d = torch.from_numpy(s).to(dev), torch.from_numpy(mu).to(dev)
    g_d = torch.from_numpy(rng.standard_normal(n).astype(np.float32)).to(dev)
    out = {}
    for split in (0, 256):
        ctx.set_split(split)
        out[split] = [t.double().cpu().numpy() for t in (
            ctx.winding(mu_d, 0.002), ctx.adjoint(s_d, 0.002), ctx.gradient(mu_d, 0.002))]
        if split:
            st = ctx.stats()
            assert st["n_tasks"] >= 3 * st["n_groups"]  # the walks are cut
    ctx.close()
    P = x.double().cpu().numpy()
    dv = P[:, None] - P[None]
    r = np.linalg.norm(dv, axis=-1)
    np.fill_diagonal(r, np.inf)
    k = 1 / (4 * np.pi)
    s64, mu64 = np.abs(s.astype(np.float64)), np.linalg.norm(mu.astype(np.float64), axis=1)
    mags = [(k * mu64 / r**2).sum(1), (k * s64 / r**2).sum(1)[:, None],
            (4 * k * mu64 / r**3).sum(1)[:, None]]
    for name, a, b, m in zip(("A", "AT", "G"), out[0], out[256], mags):
        bound = 2.0**-23 * np.abs(a) + len(rows) * 2.0**-53 * m
        bad = np.abs(a - b) > bound
        assert not bad.any(), (name, int(bad.sum()), bad.size)
