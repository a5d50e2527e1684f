"""A solve between two of its convergence tests (every 16 iterations): it goes on
to the next test while the residual is above rounding, however coarse the
tolerance, and reports the iterations that it ran."""
import numpy as np
import pytest

from paper_2005_05899_amd import meshgen as mg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cube():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import step
    from paper_2005_05899_amd import lesasm
    c = mg.periodic_tg_case(8)
    m = lesasm.Mesh.from_arrays(c.mesh, c.vreman_c)
    yield torch, lesasm, c, m, step.laplacian(c.mesh), c.mesh.field_coords()
    m.close()


@pytest.mark.parametrize("rtol", [0.5, 1e-2, 1e-3])
def test_coarse_tolerance_runs_to_its_test(cube, rtol):
    # one mode and a little noise: the oracle's residual is 5e-4 after one
    # iteration, above 1e-12 until the 16th and 1.3e-12 after it (bar 1e-10);
    # solutions to 1e-9 of the largest entry, as in test_gpu_cg_ends.py
    from oracle import cg
    torch, lesasm, c, m, K, x = cube
    b = np.cos(x[:, 0]) + 1e-4 * np.random.default_rng(3).standard_normal(len(x))
    st = lesasm.Stepper(m, c.nu, 1e-3, rtol=rtol, maxit=100)
    got = m.to_user(st.pressure_solve(m.to_internal(torch.from_numpy(b).cuda()))).cpu().numpy()
    it, res = st.stats()
    st.close()
    want = cg.jacobi_pcg(K, b, 16, rtol=0.0)[0]
    assert it == 16 and res <= 1e-10
    assert np.abs(got - want).max() <= 1e-9 * np.abs(want).max()


@pytest.mark.parametrize("modes", [1, 2, 3, 4])
def test_reported_iterations_are_those_run(cube, modes):
    # as many distinct eigenvalues as modes: CG ends after that many iterations
    # (the oracle's residual is then below 6e-15, and below 5e-16 one iteration
    # on), long before its first test
    torch, lesasm, c, m, K, x = cube
    parts = [np.cos(x[:, 0]), np.cos(2 * x[:, 1]), np.cos(x[:, 0] + x[:, 1]), np.cos(3 * x[:, 2])]
    b = m.to_internal(torch.from_numpy(sum(parts[:modes])).cuda())
    st = lesasm.Stepper(m, c.nu, 1e-3)
    for _ in range(2):
        st.pressure_solve(b)
        it, res = st.stats()
        assert modes <= it <= modes + 1 and res <= 1e-14
    st.close()
    # and after one iteration less a solve reports a residual above rounding
    if modes > 1:
        st = lesasm.Stepper(m, c.nu, 1e-3, maxit=modes - 1)
        st.pressure_solve(b)
        assert st.stats()[0] == modes - 1 and st.stats()[1] > 1e-2
        st.close()


def test_many_tests_before_the_last(cube):
    # six tests with iterations queued behind each: the oracle's residual is
    # 3.3e-10 after 80 iterations and 3.0e-12 after 96.  One ulp in the matrix
    # (its values are summed by atomics) moves these by up to 8.4e-14, hence the
    # absolute 1e-12 on the residual
    from oracle import cg, step
    torch, lesasm = cube[:2]
    c = mg.small_hybrid_case(nx=11, ny=9, layers=[(mg.HEX08, 2), (mg.PEN06, 2), (mg.TET04, 2), (mg.PYR05, 1)], seed=8)
    m = lesasm.Mesh.from_arrays(c.mesh, c.vreman_c)
    K = step.laplacian(c.mesh)
    b = np.random.default_rng(5).standard_normal(m.n_field_nodes)
    bd = m.to_internal(torch.from_numpy(b).cuda())
    st = lesasm.Stepper(m, c.nu, 1e-3, rtol=1e-10, maxit=5000)
    want, _, res_o = cg.jacobi_pcg(K, b, 96, rtol=0.0)
    for _ in range(2):
        x = m.to_user(st.pressure_solve(bd)).cpu().numpy()
        it, res = st.stats()
        assert it == 96 and res <= 1e-10 and abs(res - res_o) <= 1e-12
        assert np.abs(x - want).max() <= 1e-9 * np.abs(want).max()
    st.close()
    m.close()
