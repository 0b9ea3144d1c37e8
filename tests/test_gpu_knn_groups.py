"""Nearest neighbours at the edges of the search's groups and stack: fewer
points than neighbours, more coincident points than a group holds, isolated
points far from a dense patch, thin lines, children's offsets wider than 16
bits, and clouds of a batch.  Against every distance of sampled points in FP64.

Bound: the search orders by FP32 distances of FP32 points, each within
3 * 2^-24 of the true one relative to the coordinates' differences squared, so
the k-th distance differs from the exact one by less than 1e-6 of it (plus
1e-12 for coincident points); the neighbours themselves may swap within that.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _clouds(kind, rng):
    if kind == "few":
        return [rng.standard_normal((n, 3)) for n in (3, 5, 16, 17, 18, 33, 64, 65)]
    if kind == "coincident":
        p = rng.standard_normal((500, 3))
        p[100:300] = p[7]
        return [p]
    if kind == "isolated":
        return [np.concatenate([0.01 * rng.standard_normal((3000, 3)) + 0.3,
                                rng.uniform(-1, 1, (40, 3)), 0.001 * rng.standard_normal((900, 3)) - 0.5])]
    if kind == "line":
        t = np.linspace(0, 1, 5000)
        return [np.stack([t, t * t, 1e-3 * np.sin(40 * t)], 1)]
    p = rng.standard_normal((150000, 3))
    return [p / np.linalg.norm(p, axis=1, keepdims=True), rng.uniform(-1, 1, (1000, 3))]


@pytest.mark.parametrize("kind,leaf_cap", [("few", 1), ("coincident", 1), ("isolated", 1),
                                           ("isolated", 8), ("line", 1), ("wide", 1)])
def test_neighbours_at_group_edges(kind, leaf_cap):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16634_amd as w
    w.load_library()
    print(f"[case] knn groups {kind} {leaf_cap}", flush=True)
    rng = np.random.default_rng(5)
    clouds = [c.astype(np.float32) for c in _clouds(kind, rng)]
    offs = np.concatenate([[0], np.cumsum([len(c) for c in clouds])])
    ctx = w.Context(0)
    pts = torch.from_numpy(np.concatenate(clouds)).to("cuda:0")
    offd = [int(o) for o in offs]
    if len(clouds) > 1:
        x = ctx.normalize_batched(pts, offd)[0]
        ctx.build_batched(x, offd, leaf_cap=leaf_cap)
    else:
        x = ctx.normalize(pts)[0]
        ctx.build(x, leaf_cap=leaf_cap)
    P = x.cpu().numpy().astype(np.float64)
    nbr = ctx.features(with_neighbours=True)[1].cpu().numpy()
    for a, b in zip(offs[:-1], offs[1:]):
        k = min(16, b - a - 1)
        rows = np.arange(a, b) if b - a <= 4000 else rng.choice(np.arange(a, b), 400, replace=False)
        for i in rows:
            d = ((P[a:b] - P[i]) ** 2).sum(1)
            d[i - a] = np.inf
            want = np.sort(d)[:k]
            got = nbr[i, :k]
            assert (nbr[i, k:] == -1).all()
            assert ((got >= a) & (got < b) & (got != i)).all() and len(set(got)) == k
            assert np.all(np.abs(d[got - a] - want) <= 1e-6 * want + 1e-12), (i, d[got - a], want)
    ctx.close()
