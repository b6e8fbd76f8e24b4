"""A finest level that is streamed keeps its rows in tiles however a call runs: an operator set up by
one way of calling (streamed; launches per pass in a workspace without the mailbox; recorded into a
graph) and reused by another gives the same correction bit for bit."""
import ctypes as C

import pytest
import torch

from swe_workloads import wedge_problem
from test_gpu_resident2d import _operator

pytestmark = pytest.mark.gpu

# exact tiles; a last row of tiles of four cells, FP64; ragged, and one more tile row than full ones, FP32
GRIDS = [(768, 384, 8, 0), (64, 2112, 7, 0), (128, 4224, 8, 1)]


def _cycle(s, nbytes, J, rhs, dU, setup):
    from paper_2505_10857_amd import _abi as A
    A.check(s.L.nmg_mg_vcycle(C.byref(s.dev.desc), C.byref(s.params), C.c_void_p(s.workspace().data_ptr()), nbytes,
                              C.c_void_p(J.data_ptr()), C.c_void_p(rhs.data_ptr()), C.c_void_p(dU.data_ptr()), setup,
                              C.c_void_p(torch.cuda.current_stream().cuda_stream)))


@pytest.mark.parametrize("nx,ny,levels,prec", GRIDS)
def test_set_up_one_way_and_reused_another(nx, ny, levels, prec):
    from paper_2505_10857_amd import Solver2D
    s = Solver2D(wedge_problem(nx, ny, levels=levels), device="cuda", precision=prec, nu1=2, nu2=1)
    J, rhs = _operator(nx, ny, 9, prec)
    full = s.workspace().numel()
    out = []
    for first, second in ((full, full), (full, full - 1), (full - 1, full), (full - 1, full - 1)):
        s.workspace().fill_(0x5a)
        dU = 0.01 * rhs
        _cycle(s, first, J, rhs, dU, 1)
        _cycle(s, second, J, rhs, dU, 0)
        out.append(dU)
    # the reuse recorded, and replayed after an eager set-up of another operator
    dU = 0.01 * rhs
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    _cycle(s, full, J * 1.5, rhs, dU, 1)
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=side):
        _cycle(s, full, J, rhs, dU, 0)
    for _ in range(2):
        dU.copy_(0.01 * rhs)
        _cycle(s, full, J, rhs, dU, 1)
        g.replay()
        torch.cuda.synchronize()
        out.append(dU.clone())
    # the other form of a launched pass
    s.params.schedule = 1
    dU = 0.01 * rhs
    _cycle(s, full - 1, J, rhs, dU, 1)
    _cycle(s, full - 1, J, rhs, dU, 0)
    out.append(dU)
    assert torch.isfinite(out[0]).all()
    for v in out[1:]:
        assert torch.equal(out[0], v)
