"""The warm-start network at the edges of its tiles (32 rows per wavefront, 128
per workgroup, 256 workgroups of partial gradients): outputs and gradients
against the oracle's network in the same precision (BF16 operands), and a
feature array that is not 16-byte aligned gives the same bits.

Bounds: the device rounds the same FP32 values to BF16, except that its FP32
sums differ from the oracle's FP64 ones by a few 2^-24 and so may round a
hidden activation to the neighbouring BF16 value (2^-8 of it) when it lies on
a boundary (about one activation in 10^4).  One such activation in 64, each
with a weight of order 1/8 of the output's, moves an output by about 2^-8 / 8;
1e-2 of the RMS output and of the gradient's norm bound it with room for a row
whose output is small.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 31, 32, 33, 127, 128, 129, 4095, 32768, 33000])
def test_network_at_tile_edges(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16634_amd as w
    from oracle import mlp as om
    from paper_2405_16634_amd import warmstart
    w.load_library()
    print(f"[case] mlp tiles n={n}", flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n)
    p = warmstart.init_params(3)
    p = (p + 0.05 * rng.standard_normal(p.size)).astype(np.float32)
    X = rng.standard_normal((n, 48)).astype(np.float32)
    L = rng.standard_normal((n, 3))
    L = (L / np.linalg.norm(L, axis=1, keepdims=True)).astype(np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ctx = w.Context(0)
    pd, Ld = t(p), t(L)
    res = []
    for shift in (0, 1):  # a view one float into a buffer: 4-byte aligned
        buf = torch.empty(n * 48 + 1, device=dev)
        Xd = buf[shift:shift + n * 48].view(n, 48)
        Xd.copy_(t(X))
        out, grad = torch.empty(n, 3, device=dev), torch.empty(w.MLP_PARAMS, device=dev)
        w.wnnc_mlp_forward(ctx.handle, pd, Xd, out)
        loss = w.wnnc_mlp_grad(ctx.handle, pd, Xd, Ld, grad)
        res.append((out.cpu().numpy(), grad.cpu().numpy(), loss))
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])
    assert res[0][2] == res[1][2]
    out, grad, loss = res[0]
    y = om.forward(p.astype(np.float64), X.astype(np.float64))[2]
    ref = y / np.linalg.norm(y, axis=1, keepdims=True)
    assert np.sqrt(((out - ref) ** 2).sum(1).mean()) <= 1e-2
    ref_loss, ref_grad = om.loss_grad(p.astype(np.float64), X.astype(np.float64), L.astype(np.float64))
    assert loss == pytest.approx(ref_loss, abs=1e-3)
    assert np.linalg.norm(grad - ref_grad) <= 1e-2 * np.linalg.norm(ref_grad)
    ctx.close()
