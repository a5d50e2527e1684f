"""Training on the last, partly filled tile of samples (16 a wavefront, 64 a
workgroup, 256 workgroups a round): samples past the end take no part in any
sum, and each one before it does."""
import numpy as np
import pytest

from oracle import mlp as omlp
from tests.test_gpu_mlp_tiles import U, reference


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 15, 16, 63, 64, 65, 200])
def test_overflow_of_no_sample_reaches_the_gradients(torch_cuda, n):
    # unit 0 of the first layer is far below zero for every sample (input 0 is 1)
    # but far above it without inputs, where the second layer overflows; the
    # network without that unit gives the same sums bit for bit
    from paper_2005_05899_amd import lesasm
    torch = torch_cuda
    rng = np.random.default_rng(n)
    p = {k: v + 0.05 * rng.standard_normal(v.shape) for k, v in omlp.init_params(71).items()}
    p["b2"] = np.abs(p["b2"]) + 0.1
    x = rng.standard_normal((n, 10)).astype(np.float32)
    x[:, 0] = 1.0
    t = rng.standard_normal((n, 6)).astype(np.float32)
    got = []
    for w, b, w2 in ((-1e30, 5e29, 1e20), (-1.0, -1.0, 0.0)):
        p["W1"][:, 0] = 0.0
        p["W1"][0, 0], p["b1"][0], p["W2"][0] = w, b, w2
        m = lesasm.MLP(omlp.flatten(p).astype(np.float32))
        loss, grad = m.loss_grad(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda())
        got.append((float(loss), grad.cpu().numpy()))
        m.close()
    assert np.isfinite(got[0][0]) and np.isfinite(got[0][1]).all()
    assert got[0][0] == got[1][0] and np.array_equal(got[0][1], got[1][1])


# (samples, the one sample whose targets are 1e5 times the others': the loss and
# every gradient it enters are then its own, so the bars see whether it is there)
WEIGHTY = [(n, s) for n in (1, 15, 17, 63, 64, 65, 129, 1000, 16384, 16385, 40001)
           for s in sorted({0, n - 1, (n - 1) // 64 * 64, (n - 1) // 16 * 16, 16383, 16384, 32768}) if s < n]


def weighty(n, s):
    rng = np.random.default_rng(n)
    p = {k: (v + 0.05 * rng.standard_normal(v.shape)).astype(np.float32).astype(np.float64)
         for k, v in omlp.init_params(61).items()}
    x = rng.standard_normal((n + n // 20 + 50, 10)).astype(np.float32).astype(np.float64)
    a1 = x @ p["W1"] + p["b1"]  # masks agree: as in test_gpu_mlp_tiles.py
    a2 = np.maximum(a1, 0) @ p["W2"] + p["b2"]
    x = x[(np.abs(a1).min(1) > 1e-4) & (np.abs(a2).min(1) > 1e-4)][:n]
    assert len(x) == n
    t = rng.standard_normal((n, 6)).astype(np.float32).astype(np.float64)
    t[s] *= 1e5
    t = t.astype(np.float32).astype(np.float64)
    # bars: as in test_gpu_mlp_tiles.py
    k = (11 + 65 + 65 + 8) + (6 + 64) + 64 + -(-n // 16384) * 16 + 40
    return p, x, t, 2 * k * U


@pytest.mark.parametrize("n, s", WEIGHTY)
def test_bars_see_a_lost_sample(n, s):
    p, x, t, bar = weighty(n, s)
    (_, loss, g), (_, la, ga) = reference(p, x, t)
    without, gw = 0.0, np.zeros_like(g)
    if n > 1:
        rest = np.arange(n) != s
        _, without, gw = reference(p, x[rest], t[rest])[0]
        without, gw = without * (n - 1) / n, gw * (n - 1) / n
    assert abs(without - loss) > 100 * bar * la
    assert (np.abs(gw - g) > 100 * bar * ga).any()


@pytest.mark.gpu
@pytest.mark.parametrize("n, s", WEIGHTY)
def test_every_sample_counts(torch_cuda, n, s):
    from paper_2005_05899_amd import lesasm
    torch = torch_cuda
    p, x, t, bar = weighty(n, s)
    (_, loss, g), (_, la, ga) = reference(p, x, t)
    m = lesasm.MLP(omlp.flatten(p).astype(np.float32))
    got_l, got_g = m.loss_grad(*(torch.from_numpy(v.astype(np.float32)).cuda() for v in (x, t)))
    got_g = got_g.cpu().numpy().astype(np.float64)
    m.close()
    assert abs(float(got_l) - loss) <= bar * la
    assert (np.abs(got_g - g) <= bar * ga).all()
