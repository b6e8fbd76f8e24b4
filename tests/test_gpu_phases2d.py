"""Newton steps whose smoothing phases have few passes or none, as cooperative launches and (in a
workspace without the mailbox) as separate launches: the same operations on the same values, so
equal bit for bit.  The three cycles of a step run a level's post-smoothing and the next
pre-smoothing in one phase."""
import ctypes as C

import pytest
import torch

from swe_workloads import wedge_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("jac", [9, 21])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nu1,nu2", [(0, 0), (0, 1), (1, 0), (1, 1), (1, 2)])
@pytest.mark.parametrize("nx,ny,levels", [(64, 32, 4), (320, 96, 6)])
def test_short_phases_equal_separate_launches(nx, ny, levels, nu1, nu2, prec, jac):
    from paper_2505_10857_amd import Solver2D
    s = Solver2D(wedge_problem(nx, ny, levels=levels, seed=7), device="cuda", precision=prec, jac=jac, nu1=nu1, nu2=nu2)
    ws = s.workspace()
    out = []
    for nbytes in (ws.numel(), ws.numel() - 1):
        ws.fill_(0x5a)
        U = s.state()
        args = (C.byref(s.dev.desc), C.byref(s.params), C.c_void_p(ws.data_ptr()), nbytes, C.c_void_p(U.data_ptr()))
        stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert s.L.nmg_newton2d_begin(*args, stream) == 0
        assert s.L.nmg_newton2d_steps(*args, 2, None, stream) == 0
        out.append(U)
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1])
