"""The split at the edges of its tiles: rows of 16 lanes, runs across wavefronts
and workgroups, one scan tile and many, and target tables in kernel arguments
and in memory, bit for bit against the oracle; and centroids of meshes whose
neighbouring elements differ in node count."""
import numpy as np
import pytest

from oracle import partition as op

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("level", [1, 3, 4, 5, 7, 8])
@pytest.mark.parametrize("n, parts, lam", [(1, 1, False), (15, 2, True), (17, 3, False), (64, 5, True), (257, 256, True),
                                           (1000, 257, True), (5000, 300, False), (70000, 37, True)])
def test_parts_equal_the_oracles(torch_cuda, n, parts, lam, level):
    from paper_2005_05899_amd import lesasm
    torch = torch_cuda
    rng = np.random.default_rng(n + level)
    c = np.cumsum(rng.uniform(-0.01, 0.011, (n, 3)), axis=0)  # a walk: long runs of equal and adjacent bins
    c[rng.integers(0, n, n // 7)] = rng.uniform(c.min(), c.max() + 1e-9, (n // 7, 3))
    w = rng.integers(0, 2 ** 31 - 1, n).astype(np.int32)
    lm = rng.uniform(0.0, 2.0, parts) if lam else None
    if lam:
        lm *= parts / lm.sum()
    for wt in (w, None):
        got = lesasm.sfc_partition(torch.from_numpy(c).cuda(), None if wt is None else torch.from_numpy(wt).cuda(), parts,
                                   lm, level)
        want, _, _ = op.sfc_partition(c, wt, parts, lam=lm, level=level)
        assert np.array_equal(got.cpu().numpy(), want)


def test_centroids_of_mixed_neighbours(torch_cuda):
    from paper_2005_05899_amd import lesasm
    torch = torch_cuda
    rng = np.random.default_rng(3)
    k = rng.choice([4, 5, 6, 8], 20000)
    off = np.concatenate([[0], np.cumsum(k)]).astype(np.int64)
    conn = rng.integers(0, 9000, off[-1]).astype(np.int32)
    xyz = rng.standard_normal((9000, 3))
    cen, w = lesasm.element_centroids(*(torch.from_numpy(v).cuda() for v in (off, conn, xyz)))
    s = np.zeros((len(k), 3))
    for a in range(8):
        has = a < k
        s[has] += xyz[conn[off[:-1][has] + a]]
    assert np.array_equal(cen.cpu().numpy(), s / k[:, None])
    assert np.array_equal(w.cpu().numpy(), np.where(k == 5, 8, k))
