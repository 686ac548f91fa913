"""GPU: the products of the adjoint against the oracle's tangent, each group of inputs (U, its derivatives, b, b_x, b_y) by itself, so
that none hides behind a larger one. Grids on both sides of every edge of the interface reverse's patches (61 or 29 interfaces
along x, 13 along y, 4 lines in y) and of the rule for a wavefront per field (507 and 595 to 785 patches for 256 CUs)."""
import numpy as np
import pytest

import test_gpu_adjoint as base

pytestmark = pytest.mark.gpu

SHAPES = [(4, 4), (12, 5), (13, 61), (28, 12), (29, 27), (60, 13), (61, 14), (59, 25), (122, 26), (123, 9), (121, 130),
          (182, 77), (184, 78), (181, 104), (182, 103), (183, 105)]


@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_products_by_group(oracle_mod, inputs_mod, nx, ny, bc):
    import torch

    from paper_2208_01260_amd.solver import Solver

    O = oracle_mod
    pr = inputs_mod.paper_accuracy_2d(max(nx, ny))  # depth about 10, moving; a window of it
    cut = lambda a: np.ascontiguousarray(a[..., :ny, :nx])  # noqa: E731
    pr.nx, pr.ny, pr.bc = nx, ny, bc
    pr.state, pr.b, pr.bx, pr.by = (cut(a) for a in (pr.state, pr.b, pr.bx, pr.by))
    p = O.params_of(pr)
    rng = np.random.default_rng(1000 * nx + ny)
    ax, ay = O.alpha(p, pr.state, pr.b, pr.bx, pr.by)
    al = (1.05 * ax, 1.05 * ay)
    rbar, mbar = rng.standard_normal(pr.state.shape), rng.standard_normal((6,) + pr.b.shape)
    with Solver.from_problem(pr) as s:
        st, rb, mb = (base.dev(torch, a) for a in (pr.state, rbar, mbar))
        g = [base.host(a) for a in s.rhs_vjp(st, rb, al)]
        lim = [base.host(a) for a in s.limit_vjp(st, mb)]
    ds, db, dbx, dby = base.directions(pr, rng)
    dU, dD, z, zs = ds.copy(), ds.copy(), np.zeros_like(pr.b), np.zeros_like(pr.state)
    dU[3:], dD[:3] = 0.0, 0.0
    for name, d in (("U", (dU, z, z, z)), ("D", (dD, z, z, z)), ("b", (zs, db, z, z)), ("bx", (zs, z, dbx, z)),
                    ("by", (zs, z, z, dby))):
        def tangent(x):
            _, dR = O.rhs_jvp(p, x, d[0], pr.b, pr.bx, pr.by, d[1], d[2], d[3], al[0], al[1])
            return float(np.sum(rbar * dR))

        base.check_dot(f"rhs {nx}x{ny} {name}", tangent, pr.state, float(sum(np.sum(a * b) for a, b in zip(g, d))))
        if name in ("bx", "by"):
            continue  # the limiter does not read the slopes

        def limited(x):
            _, dD_ = O.limit_jvp(p, x, d[0], pr.b, pr.bx, pr.by, d[1], z, z)
            return float(np.sum(mbar * dD_))

        base.check_dot(f"limit {nx}x{ny} {name}", limited, pr.state, float(sum(np.sum(a * b) for a, b in zip(lim, d[:2]))))
