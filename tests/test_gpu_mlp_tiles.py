"""Training and FP32 inference of the closure network at the edges of their
tiles (16 samples a wavefront, 64 a workgroup, 256 workgroups) against FP64.

Bars: the standard rounding bound of a chain of FP32 sums and products, k u
times the same computation on absolute values (u = 2^-24, k the operations on
the longest path).  ReLU masks have to agree for that, so samples with a
hidden pre-activation within 1e-4 of zero are left out of the inputs."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.fixture(scope="module")
def setup():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_05899_amd import lesasm
    p = omlp.init_params(61)
    rng = np.random.default_rng(62)
    p = {k: (v + 0.05 * rng.standard_normal(v.shape)).astype(np.float32).astype(np.float64) for k, v in p.items()}
    x = rng.standard_normal((44000, 10)).astype(np.float32).astype(np.float64)
    t = rng.standard_normal((len(x), 6)).astype(np.float32).astype(np.float64)
    a1 = x @ p["W1"] + p["b1"]
    a2 = np.maximum(a1, 0) @ p["W2"] + p["b2"]
    keep = (np.abs(a1).min(1) > 1e-4) & (np.abs(a2).min(1) > 1e-4)
    m = lesasm.MLP(omlp.flatten(p).astype(np.float32))
    yield torch, m, p, x[keep], t[keep]
    m.close()


def reference(p, x, t):
    """(y, loss, gradients) in FP64 and the same on absolute values."""
    out = []
    for f in (lambda v: v, np.abs):
        w1, b1, w2, b2, w3, b3 = (f(p[k]) for k in omlp.ORDER)
        ab = f is np.abs
        a1 = f(x) @ w1 + b1
        h1 = a1 if ab else np.maximum(a1, 0)
        a2 = h1 @ w2 + b2
        h2 = a2 if ab else np.maximum(a2, 0)
        y = h2 @ w3 + b3
        z = y.copy()
        z[:, :3] += (1 if ab else -1) * y[:, :3].mean(1, keepdims=True)
        r = z + f(t) if ab else z - t
        w = np.array([1.0, 1, 1, 2, 2, 2])
        loss = (w * r * r).sum() / len(x)
        dy = 2 * w * r / len(x)
        dy[:, :3] += (1 if ab else -1) * dy[:, :3].mean(1, keepdims=True)
        d2 = (dy @ w3.T) * (1 if ab else a2 > 0)
        d1 = (d2 @ w2.T) * (1 if ab else a1 > 0)
        g = [f(x).T @ d1, d1.sum(0), h1.T @ d2, d2.sum(0), h2.T @ dy, dy.sum(0)]
        out.append((y, loss, np.concatenate([v.ravel() for v in g])))
    return out


@pytest.mark.parametrize("n", [1, 15, 17, 63, 64, 65, 129, 1000, 16384, 16385, 40001])
def test_loss_gradients_and_forward(setup, n):
    torch, m, p, x, t = setup
    x, t = x[:n], t[:n]
    assert len(x) == n
    xd, td = (torch.from_numpy(np.ascontiguousarray(v, np.float32)).cuda() for v in (x, t))
    (y, loss, g), (ya, la, ga) = reference(p, x, t)
    print(f"  n = {n}", flush=True)
    got_y = m.forward_f32(xd).cpu().numpy().astype(np.float64)
    assert (np.abs(got_y - y) <= (11 + 65 + 65) * U * ya).all()
    got_l, got_g = m.loss_grad(xd, td)
    k = (11 + 65 + 65 + 8) + (6 + 64) + 64 + -(-n // 16384) * 16 + 40  # forward, back, a tile, a workgroup's tiles, the sum over workgroups
    assert abs(float(got_l) - loss) <= 2 * k * U * la
    got_g = got_g.cpu().numpy().astype(np.float64)
    assert (np.abs(got_g - g) <= 2 * k * U * ga).all()
    again = m.loss_grad(xd, td)[1].cpu().numpy()
    assert np.array_equal(again, got_g.astype(np.float32))  # fixed order of every sum
