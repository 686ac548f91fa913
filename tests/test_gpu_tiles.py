"""GPU: the tile of a stage changes no bit of any result. Grids that take workgroups of 1 to 8 rows
(by their size on a device of 256 CUs), the smallest, ragged and periodic ones among them, against the
marching wavefronts, which SWE_HWENO_ROWS asks for; and marches of different lengths against each other."""
import os

import pytest

pytestmark = pytest.mark.gpu

# nx, ny and the rows per workgroup on 256 CUs (tiles of 60 columns; 0 = marching wavefronts)
SHAPES = [(4, 4, 1), (61, 47, 1), (59, 256, 1), (61, 129, 2), (130, 171, 3), (180, 339, 4), (240, 319, 5), (300, 301, 6),
          (299, 357, 7), (300, 408, 8), (300, 409, 0)]


def _solver(pr, rows, dtype, **kw):
    from paper_2208_01260_amd.solver import Solver

    old = os.environ.pop("SWE_HWENO_ROWS", None)
    try:
        if rows:
            os.environ["SWE_HWENO_ROWS"] = str(rows)
        return Solver.from_problem(pr, dtype=dtype, **kw)
    finally:
        os.environ.pop("SWE_HWENO_ROWS", None)
        if old is not None:
            os.environ["SWE_HWENO_ROWS"] = old


@pytest.mark.parametrize("nx,ny,rows", SHAPES)
def test_small_tiles_give_the_bits_of_marches(nx, ny, rows):
    import torch

    from paper_2208_01260_amd import inputs
    from paper_2208_01260_amd._lib import NO_LIMITER

    dtype = torch.float64
    pr = inputs.c3_2d(nx, ny=ny)  # walls, a dam break
    if (nx + ny) % 2:
        pr.bc = (0, 0)  # periodic
    flags = NO_LIMITER if nx % 3 == 0 and ny % 2 else 0
    st = torch.from_numpy(pr.state).cuda().to(dtype)
    out = []
    for force in (0, 16, 5):
        with _solver(pr, force, dtype, flags=flags) as s:
            if not force and torch.cuda.get_device_properties(0).multi_processor_count == 256:
                assert rows == 0 or s.tile()[1] == rows
            r = s.rhs(st)
            given = s.rhs(st, alpha=(7.0, 9.0))
            x = st.clone()
            t = s.run(x, nsteps=4)
            y = st.clone()
            s.step(y, dt=1e-5)
            out.append((r, given, x, y, t))
    for o in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(o[:4], out[0][:4])) and o[4] == out[0][4], (nx, ny)


def test_small_tile_reports_dry_and_nonfinite():
    import torch

    from paper_2208_01260_amd import inputs
    from paper_2208_01260_amd.solver import Solver, SweError

    pr = inputs.c2_2d(61, "smooth", ny=47)
    for bad, code in ((-5.0, -4), (float("nan"), -5)):
        st = torch.from_numpy(pr.state).cuda()
        st[0, 46, 60] = bad
        with Solver.from_problem(pr) as s:
            s.rhs(st, alpha=(5.0, 5.0))
            with pytest.raises(SweError) as e:
                s.sync()
            assert e.value.code in ((code,) if code == -5 else (-4, -5))
            with pytest.raises(SweError):
                s.run(st.clone(), nsteps=2)
