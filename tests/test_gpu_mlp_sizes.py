"""The perceptron's products at the edges of their tiling (32 x 32 tiles, 16-deep
steps dealt to eight waves, rows that are not 16-byte aligned, one training row,
outputs past one workgroup's loss sum) against the FP64 reference at the same
bf16 weights.

Tolerance: each product carries its FP32 operands to 2^-16 and accumulates K
terms in FP32; through at most three layers with tanh slopes below one and
unit-size rows of weights the relative error stays below 2e-4 of the largest
entry (the bound of the gradient test at smaller sizes)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import mlp as M

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("widths,batch", [((1, 1), 1), ((5, 33, 7), 1), ((8, 16, 32), 33), ((3, 600, 31), 31),
                                          ((16, 1030, 24), 40), ((7, 129, 257, 65), 65), ((2, 24, 2050), 33),
                                          ((4, 136, 96), 300)])
def test_mlp_sizes(widths, batch):
    print("CASE mlp sizes", widths, batch, flush=True)
    from paper_1510_03330_amd.warmstart import MLP
    net = MLP(widths, DEV, seed=1)
    rng = np.random.default_rng(5)
    p = np.concatenate([np.concatenate([(rng.standard_normal(o * i) / np.sqrt(i)), 0.1 * rng.standard_normal(o)])
                        for i, o in zip(widths[:-1], widths[1:])]).astype(np.float32)
    net.set_params(torch.from_numpy(p))
    x = rng.standard_normal((batch, widths[0])).astype(np.float32)
    t = rng.standard_normal((batch, widths[-1])).astype(np.float32)
    X, Tt = torch.from_numpy(x).to(DEV), torch.from_numpy(t).to(DEV)
    acts, out = net.forward(X)
    ref = M.forward(p.astype(np.float64), widths, x.astype(np.float64))
    got = acts.cpu().numpy().astype(np.float64)
    off = 0
    for r in ref:
        a = got[off:off + r.size].reshape(r.shape)
        assert np.max(np.abs(a - r)) < 2e-4 * max(1e-3, np.max(np.abs(r)))
        off += r.size
    loss = net.backward(X, acts, Tt)
    lref, gref = M.loss_and_grad(p.astype(np.float64), widths, x.astype(np.float64), t.astype(np.float64))
    assert abs(float(loss.item()) - lref) < 1e-4 * lref
    assert np.max(np.abs(net.g.cpu().numpy() - gref)) < 2e-4 * np.max(np.abs(gref))
