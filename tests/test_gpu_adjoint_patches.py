"""GPU: the patches of the adjoint's interface reverse. Grids whose n + 1 interfaces end one before, at and one after a
patch's edge (61 or 29 along x, 13 along y, 4 lines in y), the smallest grids among them: the vector-Jacobian product
of the right-hand side and a run's gradient against directional derivatives by the library's own forward maps (the transpose
identity with central differences)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(4, 4), (12, 5), (13, 61), (28, 12), (29, 27), (60, 13), (61, 14), (59, 25), (122, 26), (123, 9), (121, 130)]


@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (0, 1)])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_rhs_vjp_transpose_identity(nx, ny, bc):
    import torch

    from paper_2208_01260_amd import inputs
    from paper_2208_01260_amd.solver import Solver

    rng = np.random.default_rng(nx * 1000 + ny)
    pr = inputs.paper_accuracy_2d(max(nx, ny))  # depth about 10, moving; a window of it
    cut = lambda a: np.ascontiguousarray(a[..., :ny, :nx])  # noqa: E731
    dom, alpha = (0.0, 1.0, 0.0, 1.0), (12.0, 13.0)
    t = lambda a: torch.from_numpy(cut(a)).cuda()  # noqa: E731
    st, base = t(pr.state), [t(pr.b), t(pr.bx), t(pr.by)]
    rbar = torch.from_numpy(rng.standard_normal((9, ny, nx))).cuda()
    d = [torch.from_numpy(rng.standard_normal(x.shape)).cuda() for x in [st] + base]

    def f(eps):
        b = [x + eps * y for x, y in zip(base, d[1:])]
        with Solver(2, nx, ny, dom, *b, bc=bc) as s:
            return (s.rhs(st + eps * d[0], alpha=alpha) * rbar).sum().item(), s.rhs(st, alpha=alpha).abs().max().item()

    with Solver(2, nx, ny, dom, *base, bc=bc) as s:
        g = s.rhs_vjp(st, rbar, alpha)
    adj = sum((x * y).sum().item() for x, y in zip(g, d))
    # fourth-order central differences with steps h and h / 2; their own spread bounds the truncation
    h = 1e-4
    c = [(8 * (f(x)[0] - f(-x)[0]) - (f(2 * x)[0] - f(-2 * x)[0])) / (12 * x) for x in (h, h / 2)]
    scale = sum((x.abs() * y.abs()).sum().item() for x, y in zip(g, d))
    # the rounding of a difference quotient: the forward's sum of |R| terms at 1e-16 over the step
    rounding = 4e-16 * f(0.0)[1] * rbar.abs().sum().item() / h
    assert abs(adj - c[1]) <= 16 * abs(c[0] - c[1]) + 20 * rounding + 1e-10 * scale, (adj, c, scale)
