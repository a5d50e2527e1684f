"""Training on the last, partly filled tile of samples (16 a wavefront, 64 a
workgroup): samples past the end take no part in any sum."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


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
