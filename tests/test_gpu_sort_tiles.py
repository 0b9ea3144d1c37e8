"""The Morton sort at the edges of its tiles (64 consecutive keys per rank step,
2048 per workgroup) and of its passes (45 bits: five; 45 and ten bits of cloud
index: seven): a tree over wrongly sorted points has other neighbourhoods.

Bound: as the neighbours' distances are FP32, each sampled point's 16th
distance is within 1e-6 of the exact one, plus 1e-12.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,clouds", [(63, 1), (64, 1), (65, 1), (2047, 1), (2048, 1), (2049, 1),
                                      (6145, 1), (40, 600), (5000, 3)])
def test_sorted_neighbourhoods(n, clouds):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16634_amd as w
    w.load_library()
    print(f"[case] sort tiles n={n} clouds={clouds}", flush=True)
    rng = np.random.default_rng(n)
    pts = rng.standard_normal((n * clouds, 3)).astype(np.float32)
    offs = [n * c for c in range(clouds + 1)]
    ctx = w.Context(0)
    t = torch.from_numpy(pts).to("cuda:0")
    if clouds > 1:
        x = ctx.normalize_batched(t, offs)[0]
        ctx.build_batched(x, offs)
    else:
        x = ctx.normalize(t)[0]
        ctx.build(x)
    P = x.cpu().numpy().astype(np.float64)
    nbr = ctx.features(with_neighbours=True)[1].cpu().numpy()
    for i in rng.choice(n * clouds, min(n * clouds, 500), replace=False):
        a = i // n * n
        d = ((P[a:a + n] - P[i]) ** 2).sum(1)
        d[i - a] = np.inf
        want, got = np.sort(d)[:16], nbr[i]
        assert ((got >= a) & (got < a + n) & (got != i)).all() and len(set(got)) == 16
        assert np.all(np.abs(d[got - a] - want) <= 1e-6 * want + 1e-12)
    ctx.close()
