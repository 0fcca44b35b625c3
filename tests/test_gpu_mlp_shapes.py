"""The perceptron's products at the edges of their tiles (32 x 32 outputs, k
steps of 32 split over four wavefronts, fragments of 8): loss, gradients and
forward pass against the FP64 oracle, in place for one layer, and into the
caller's gradient array or none."""
import numpy as np
import pytest

from oracle import mlp as om

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _setup(sizes, batch, seed=17):
    import paper_2301_04869_amd as R
    Ws, bs = om.init_params(sizes, seed)
    rng = np.random.default_rng(seed)
    bs = [rng.normal(0.0, 0.1, b.shape) for b in bs]
    p32 = np.concatenate([np.concatenate([W.ravel(), b]) for W, b in zip(Ws, bs)]).astype(np.float32)
    X = rng.normal(size=(batch, sizes[0])).astype(np.float32)
    # targets at a distance from the outputs: no cancellation in y - t
    far = rng.uniform(0.5, 1.5, (batch, sizes[-1])) * rng.choice([-1.0, 1.0], (batch, sizes[-1]))
    T = (om.forward(Ws, bs, X.astype(np.float64))[0] + far).astype(np.float32)
    m = R.Mlp(sizes, batch)
    dev = lambda a: torch.tensor(a, device="cuda")  # noqa: E731
    m.set_params(dev(p32))
    return m, Ws, bs, X, T, dev


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("sizes,batch", [
    ([1, 1], 1), ([9, 6], 33), ([7, 33, 5], 1), ([8, 32, 31], 31), ([33, 65, 40, 3], 32), ([129, 31, 97], 33),
    ([300, 513, 70], 65), ([257, 130, 225], 130)])
def test_gradients_and_forward(sizes, batch):
    m, Ws, bs, X, T, dev = _setup(sizes, batch)
    buf = torch.full((m.n_params + 1,), 7.0, dtype=torch.float32, device="cuda")
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    m.gradients(dev(X), dev(T), buf[:-1], loss)
    y, ys = (torch.zeros(batch, sizes[-1], dtype=torch.float32, device="cuda") for _ in range(2))
    # the input one float past a 16-byte boundary
    xu = torch.zeros(X.size + 1, dtype=torch.float32, device="cuda")[1:].view(X.shape)
    xu.copy_(dev(X))
    m.forward(xu, y)
    m.forward_static(xu, ys)
    loss2 = torch.zeros(1, dtype=torch.float32, device="cuda")
    m.gradients(xu, dev(T), None, loss2)
    torch.cuda.synchronize()
    lo, gW, gb = om.loss_and_grads(Ws, bs, X.astype(np.float64), T.astype(np.float64))
    got, ref = buf.cpu().numpy().astype(np.float64), np.concatenate(
        [np.concatenate([W.ravel(), b]) for W, b in zip(gW, gb)])
    # BF16 operands (unit roundoff 2^-8) through up to three layers and back:
    # a few roundoffs relative, about 5 allowed
    assert abs(float(loss.item()) - lo) <= 2e-2 * lo
    assert _rel(got[:-1], ref) <= 2e-2 and got[-1] == 7.0
    assert _rel(y.cpu().numpy(), om.forward(Ws, bs, X.astype(np.float64))[0]) <= 2e-2
    assert torch.equal(y, ys) and torch.equal(loss, loss2)


def test_one_layer_in_place():
    m, Ws, bs, X, _, dev = _setup([40, 40], 70)
    y, xy = torch.zeros(70, 40, dtype=torch.float32, device="cuda"), dev(X)
    m.forward(dev(X), y)
    m.forward(xy, xy)
    torch.cuda.synchronize()
    assert torch.equal(y, xy)
