"""Ends of the pressure CG: the iterations queued behind a convergence test must
leave no trace.  Against the oracle's CG after the same number of iterations
(bar 1e-9 of the largest entry, as for the iterates in test_gpu_step.py)."""
import numpy as np
import pytest

from paper_2005_05899_amd import meshgen as mg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import step
    from paper_2005_05899_amd import lesasm
    c = mg.small_hybrid_case(nx=11, ny=9, layers=[(mg.HEX08, 2), (mg.PEN06, 2), (mg.TET04, 2), (mg.PYR05, 1)], seed=8)
    m = lesasm.Mesh.from_arrays(c.mesh, c.vreman_c)
    yield torch, lesasm, c, m, step.laplacian(c.mesh)
    m.close()


@pytest.mark.parametrize("rtol, maxit", [(0.5, 100), (1e-3, 100), (1e-6, 100), (1e-6, 17), (1e-300, 1), (1e-300, 15),
                                         (1e-300, 16), (1e-300, 18), (1e-300, 33)])
def test_stops_after_the_tested_iteration(setup, rtol, maxit):
    from oracle import cg
    torch, lesasm, c, m, K = setup
    b = np.random.default_rng(5).standard_normal(m.n_field_nodes)
    bd = m.to_internal(torch.from_numpy(b).cuda())
    st = lesasm.Stepper(m, c.nu, 1e-3, rtol=rtol, maxit=maxit)
    for _ in range(2):
        x = m.to_user(st.pressure_solve(bd)).cpu().numpy()
        it, res = st.stats()
        assert it == maxit or (it % 16 == 0 and res <= rtol)
        want, _, res_o = cg.jacobi_pcg(K, b, it, rtol=0.0)
        assert np.abs(x - want).max() <= 1e-9 * np.abs(want).max()
        assert abs(res - res_o) <= 1e-6 * res_o + 1e-14
        if it > 16:  # not met at the test before
            assert cg.jacobi_pcg(K, b, (it - 1) // 16 * 16, rtol=0.0)[2] > rtol
    st.close()


def test_zero_right_hand_side_and_reuse(setup):
    torch, lesasm, c, m, K = setup
    n = m.n_field_nodes
    st = lesasm.Stepper(m, c.nu, 1e-3)
    const = torch.full((n,), 0.75, dtype=torch.float64, device="cuda")  # zero after the mean is taken off
    b = m.to_internal(torch.from_numpy(np.random.default_rng(6).standard_normal(n)).cuda())
    first = st.pressure_solve(b)
    its = st.stats()
    assert torch.count_nonzero(st.pressure_solve(const * 0)) == 0 and st.stats() == (0, 0.0)
    assert torch.equal(st.pressure_solve(b), first) and st.stats() == its
    # a captured step that met its tolerance leaves nothing that an eager solve reads
    s = torch.cuda.Stream()
    u, p = m.to_internal(torch.from_numpy(c.u).cuda()), m.to_internal(torch.from_numpy(c.p).cuda())
    torch.cuda.synchronize()
    g = lesasm.StepGraph(st, u, p, 400, s)
    g.launch(s)
    assert g.stats()[2]
    torch.cuda.synchronize()
    assert torch.equal(st.pressure_solve(b), first) and st.stats() == its
    g.close()
    st.close()


def test_periodic_solves_keep_their_accuracy(setup):
    # few distinct eigenvalues: the residual reaches rounding between two
    # tests, and the Laplacian cannot reduce its constant part
    from oracle import step
    torch, lesasm = setup[:2]
    c = mg.periodic_tg_case(8)
    m = lesasm.Mesh.from_arrays(c.mesh, c.vreman_c)
    K = step.laplacian(c.mesh)
    st = lesasm.Stepper(m, c.nu, 1e-3)
    rng = np.random.default_rng(1)
    for k in range(40):
        b = np.cos(c.mesh.field_coords() @ rng.integers(-2, 3, 3)) + 1e-3 * np.sin(c.mesh.field_coords()[:, k % 3])
        want = step.pressure_solve(K, b)
        x = m.to_user(st.pressure_solve(m.to_internal(torch.from_numpy(b).cuda()))).cpu().numpy()
        assert st.stats()[1] <= 1e-12, k
        assert np.abs(x - want).max() <= 1e-9 * np.abs(want).max(), k
    st.close()
    m.close()
