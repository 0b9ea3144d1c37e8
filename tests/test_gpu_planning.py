"""Planning of the split walks: the parts of every group's walk cover its
cloud's nodes once, whatever the cloud's size, so split walks (the parts of a
small cloud shorter than the split size, down to 16 visits) count exactly the
pairs of whole walks and agree with them at the summation-order bound of
`parity_bar.same_terms`.

The sizes are the edges of a 64-target group (1, 63, 64, 65 points), a cloud
whose parts are as short as they get, leaves of several points with coincident
copies, a huge c (every node is visited: the list of visited nodes overflows),
a tree of more than 2^16 nodes (child offsets beyond 16 bits) and a forest.
"""
import numpy as np
import pytest

import parity_bar
import synth

pytestmark = pytest.mark.gpu

CASES = {
    "one": ([1], 2.0, 1), "group-1": ([63], 2.0, 1), "group": ([64], 2.0, 1),
    "group+1": ([65], 2.0, 1), "short_parts": ([3077], 2.0, 1), "leaves": ([5000], 2.0, 8),
    "overflow": ([6000], 1e6, 1), "wide": ([60000], 2.0, 1), "forest": ([300, 1, 4096, 2500], 2.0, 1),
}


@pytest.mark.parametrize("case", list(CASES))
def test_split_walks_cover_the_tree_once(case, oracle_mod):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16634_amd as w
    w.load_library()
    sizes, c, cap = CASES[case]
    print(f"[case] planning {case}", flush=True)
    rng = np.random.default_rng(5)
    clouds = [synth.fibonacci_sphere(n, 1).points for n in sizes]
    if case == "leaves":
        clouds[0][100:120] = clouds[0][99]  # a leaf at the deepest level
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    dev = torch.device("cuda:0")
    ctx = w.Context(0)
    x, _ = ctx.normalize_batched(torch.from_numpy(np.concatenate(clouds)).to(dev), off)
    ctx.build_batched(x, off, c, 15, cap)
    mu = (synth.random_unit(rng, n) * 1e-3).astype(np.float32)
    rho = rng.standard_normal(n).astype(np.float32)
    mu_d, rho_d = torch.from_numpy(mu).to(dev), torch.from_numpy(rho).to(dev)
    res = {}
    for split in (0, 16, 256):
        ctx.set_split(split)
        ctx.set_flags(w.FLAG_COUNT_PAIRS)
        ctx.reset_stats()
        out = [ctx.winding(mu_d, 0.002).cpu().numpy(), ctx.gradient(mu_d, 0.002).cpu().numpy(),
               ctx.adjoint(rho_d, 0.002).cpu().numpy()]
        st = ctx.stats()
        ctx.set_flags(0)
        res[split] = (out, list(st["pairs"]))
        assert st["n_tasks"] >= st["n_groups"]
    xs = x.cpu().numpy().astype(np.float64)
    mags = [[], [], []]
    for k in range(len(sizes)):
        sl = slice(int(off[k]), int(off[k + 1]))
        T = oracle_mod.Tree(xs[sl], 15, cap)
        for q, (op, nu) in enumerate((("A", mu), ("G", mu), ("AT", rho))):
            mags[q].append(T.apply(op, nu[sl].astype(np.float64), 0.002, c, with_stats=True)[1])
    for split in (16, 256):
        assert res[split][1] == res[0][1], split
        for op, a, b, m in zip(("A", "G", "AT"), res[split][0], res[0][0], mags):
            parity_bar.same_terms(f"{case} split={split} {op}", a, b, np.concatenate(m))
    ctx.close()
