"""GPU: the forms of the adjoint's node pass (for 256 CUs): tiles of 8 nodes up to 512 of them, of 16 with wavefronts of their own for
the items up to 256, and of 16 without. The transpose identity of the right-hand side's and the limiter's products against
the oracle's tangent on both sides of each rule, and the same bits on a repeated call."""
import numpy as np
import pytest

import test_gpu_adjoint as base

pytestmark = pytest.mark.gpu

SHAPES = [(176, 184), (177, 184), (250, 256), (257, 250)]  # 506 and 529 tiles of 8, 256 and 272 of 16


@pytest.mark.parametrize("bc", [(0, 1), (1, 0)])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_products_against_the_oracle(oracle_mod, inputs_mod, nx, ny, bc):
    import torch

    from paper_2208_01260_amd.solver import Solver

    O = oracle_mod
    pr = inputs_mod.c3_2d(nx, ny=ny)  # a dam break
    pr.bc = bc
    p = O.params_of(pr)
    rng = np.random.default_rng(nx + ny)
    ax, ay = O.alpha(p, pr.state, pr.b, pr.bx, pr.by)
    al = (1.05 * ax, 1.05 * ay)
    rbar, mbar = rng.standard_normal(pr.state.shape), rng.standard_normal((6,) + pr.b.shape)
    with Solver.from_problem(pr) as s:
        st, rb, mb = (base.dev(torch, a) for a in (pr.state, rbar, mbar))
        g = s.rhs_vjp(st, rb, al)
        again = s.rhs_vjp(st, rb, al)
        lim = s.limit_vjp(st, mb)
    assert all(torch.equal(a, b) for a, b in zip(g, again))
    d = base.directions(pr, rng)

    def tangent(x):
        _, dR = O.rhs_jvp(p, x, d[0], pr.b, pr.bx, pr.by, d[1], d[2], d[3], al[0], al[1])
        return float(np.sum(rbar * dR))

    base.check_dot(f"rhs {nx}x{ny}", tangent, pr.state, float(sum(np.sum(base.host(a) * b) for a, b in zip(g, d))))

    def limited(x):
        _, dD = O.limit_jvp(p, x, d[0], pr.b, pr.bx, pr.by, d[1], 0 * pr.b, 0 * pr.b)
        return float(np.sum(mbar * dD))

    base.check_dot(f"limit {nx}x{ny}", limited, pr.state, float(sum(np.sum(base.host(a) * b) for a, b in zip(lim, d[:2]))))
