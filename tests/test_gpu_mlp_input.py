"""The perceptron's first product on either side of the rule that decides whether
it reads the FP32 input itself or a converted copy (at most 255 inputs and 256
tiles of 32 x 32): the two give the same bits, gradients agree with the FP64
oracle, and a wide input is not read once per column tile."""
import time

import numpy as np
import pytest

from oracle import mlp as om
from test_gpu_mlp_shapes import _rel, _setup

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("sizes,batch", [
    ([255, 256, 40], 1025),   # 33 x 8 tiles: converted; each part of 33 rows reads the input
    ([33, 2050, 7], 130),     # 5 x 65 tiles
    ([256, 64, 9], 65),       # too many inputs for either
])
def test_same_bits_whole_and_in_parts(sizes, batch):
    m, Ws, bs, X, T, dev = _setup(sizes, batch)
    x, y, yp = dev(X), *(torch.zeros(batch, sizes[-1], dtype=torch.float32, device="cuda") for _ in range(2))
    m.forward(x, y)
    for r in range(0, batch, 33):
        part = torch.zeros_like(y[r:r + 33])
        m.forward(x[r:r + 33].contiguous(), part)
        yp[r:r + 33] = part
    torch.cuda.synchronize()
    assert torch.equal(y, yp)
    assert _rel(y.cpu().numpy(), om.forward(Ws, bs, X.astype(np.float64))[0]) <= 2e-2


@pytest.mark.parametrize("sizes,batch", [([255, 256, 40], 1024), ([255, 256, 40], 1025), ([256, 33, 5], 40),
                                         ([31, 8192, 3], 32), ([31, 8193, 3], 32)])
def test_gradients_on_either_side(sizes, batch):
    m, Ws, bs, X, T, dev = _setup(sizes, batch)
    g, loss = torch.zeros(m.n_params, dtype=torch.float32, device="cuda"), torch.zeros(1, device="cuda")
    m.gradients(dev(X), dev(T), g, loss)
    torch.cuda.synchronize()
    lo, gW, gb = om.loss_and_grads(Ws, bs, X.astype(np.float64), T.astype(np.float64))
    ref = np.concatenate([np.concatenate([W.ravel(), b]) for W, b in zip(gW, gb)])
    # BF16 operands, as in test_gpu_mlp_shapes
    assert abs(float(loss.item()) - lo) <= 2e-2 * lo
    assert _rel(g.cpu().numpy().astype(np.float64), ref) <= 2e-2


def test_wide_input_is_read_once():
    """Two layers whose first is a 2000 x 2048 product cost about what that
    product alone costs (one layer, always converted); four times as much when
    every column tile read the FP32 rows."""
    def best(sizes):
        m, x, y = _setup(sizes, 32)[0], torch.randn(2048, sizes[0], device="cuda"), None
        m = type(m)(sizes, 2048)
        m.set_params(torch.randn(m.n_params, device="cuda") * 0.02)
        y = torch.zeros(2048, sizes[-1], device="cuda")
        t = []
        for _ in range(5):
            torch.cuda.synchronize()
            s = time.perf_counter()
            for _ in range(20):
                m.forward(x, y)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - s)
        return min(t)
    one, two = best([2000, 2048]), best([2000, 2048, 8])
    print(f"\n  {one / 20 * 1e6:.0f} us, with a second layer of 8 {two / 20 * 1e6:.0f} us")
    assert two <= 2.0 * one
