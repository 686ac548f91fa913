"""GPU: the two forms of the adjoint's interface reverse, a wavefront per field on grids of at most two patches per CU and one
for all fields above. The transpose identity of the right-hand side's product on both sides of the rule (507 and 595 to 785
patches for 256 CUs), with the patches' edges (61 along x, 13 along y) met and missed by one, and the same bits on a
repeated call."""
import pytest

from test_gpu_adjoint_patches import test_rhs_vjp_transpose_identity as transpose_identity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [(0, 1), (1, 0)])
@pytest.mark.parametrize("nx,ny", [(182, 77), (184, 78), (181, 104), (182, 103), (183, 105)])
def test_transpose_identity_on_both_sides(nx, ny, bc):
    transpose_identity(nx, ny, bc)


@pytest.mark.parametrize("nx,ny", [(5, 4), (96, 80), (182, 77), (183, 105)])
def test_repeated_product_is_the_same(nx, ny):
    import torch

    from paper_2208_01260_amd import inputs
    from paper_2208_01260_amd.solver import Solver

    pr = inputs.c3_2d(nx, ny=ny)
    st = torch.from_numpy(pr.state).cuda()
    rbar = torch.sin(torch.arange(st.numel(), dtype=torch.float64, device="cuda")).reshape(st.shape)
    with Solver.from_problem(pr) as s:
        first = s.rhs_vjp(st, rbar, (7.0, 9.0))
        for _ in range(5):
            assert all(torch.equal(a, b) for a, b in zip(s.rhs_vjp(st, rbar, (7.0, 9.0)), first))
