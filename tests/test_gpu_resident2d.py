"""2D levels whose smoothing phases run with the operator in registers (one cooperative launch per
phase) against the same levels as separate launches: the same operations on the same values, so
every result is equal bit for bit.  A workspace without the mailbox at its end selects the separate
launches."""
import ctypes as C

import pytest
import torch

from swe_workloads import wedge_problem

pytestmark = pytest.mark.gpu

# (nx, ny, levels, nu1, nu2): one tile to many, ragged last tiles, one pass to many per exchange,
# empty and unequal phases, the largest grid whose nine-block rows fit the registers in FP64 (a
# full tile on every compute unit) and one above it (only its coarse levels are resident)
GRIDS = [
    (40, 24, 4, 3, 2), (64, 32, 4, 20, 20), (56, 40, 4, 0, 3), (112, 80, 5, 2, 0), (160, 96, 6, 4, 5),
    (320, 96, 6, 1, 1), (512, 256, 7, 3, 3), (768, 384, 8, 1, 2),
]


def _operator(nx, ny, jac, prec, seed=5):
    from paper_2505_10857_amd import _abi as A
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    J = 0.2 * (torch.rand((jac, 3, 3, ny, nx), dtype=torch.float64, device="cuda", generator=g) - 0.5)
    for c in range(3):
        J[0, c, c] += 3.0
    dt = torch.float32 if prec == A.NMG_FP32_MG else torch.float64
    rhs = (2.0 * torch.rand((3, ny, nx), dtype=torch.float64, device="cuda", generator=g) - 1.0).to(dt)
    return J, rhs


def _vcycles(s, ws_bytes, J, rhs, cycles=2):
    from paper_2505_10857_amd import _abi as A
    ws = s.workspace()
    ws.fill_(0x5a)                  # nothing is taken from the workspace's old contents
    dU = 0.01 * rhs.clone()
    for c in range(cycles):
        A.check(s.L.nmg_mg_vcycle(C.byref(s.dev.desc), C.byref(s.params), C.c_void_p(ws.data_ptr()), ws_bytes,
                                  C.c_void_p(J.data_ptr()), C.c_void_p(rhs.data_ptr()), C.c_void_p(dU.data_ptr()),
                                  1 if c == 0 else 0, C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    return dU


@pytest.mark.parametrize("jac", [9, 21])
@pytest.mark.parametrize("prec_name", ["fp64", "fp32mg"])
@pytest.mark.parametrize("nx,ny,levels,nu1,nu2", GRIDS)
def test_resident_levels_equal_separate_launches(nx, ny, levels, nu1, nu2, prec_name, jac):
    from paper_2505_10857_amd import Solver2D, _abi as A
    prec = A.NMG_FP64 if prec_name == "fp64" else A.NMG_FP32_MG
    s = Solver2D(wedge_problem(nx, ny, levels=levels), device="cuda", precision=prec, jac=jac, nu1=nu1, nu2=nu2)
    J, rhs = _operator(nx, ny, jac, prec)
    full = s.workspace().numel()
    a = _vcycles(s, full, J, rhs)
    b = _vcycles(s, full - 1, J, rhs)
    assert torch.isfinite(a).all()
    assert torch.equal(a, b)


@pytest.mark.parametrize("prec_name", ["fp64", "fp32mg"])
def test_resident_newton_equals_separate_launches(prec_name):
    from paper_2505_10857_amd import Solver2D, _abi as A
    prec = A.NMG_FP64 if prec_name == "fp64" else A.NMG_FP32_MG
    s = Solver2D(wedge_problem(64, 32, seed=3), device="cuda", precision=prec, n_max=7)
    ws = s.workspace()
    out = []
    for nbytes in (ws.numel(), ws.numel() - 1):
        U, st = s.state(), A.nmg_stats()
        status = s.L.nmg_newton_solve(C.byref(s.dev.desc), C.byref(s.params), C.c_void_p(ws.data_ptr()), nbytes,
                                      C.c_void_p(U.data_ptr()), C.byref(st), None, 0,
                                      C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert status == A.NMG_NOT_CONVERGED
        out.append((U, st.iters, st.res))
    assert out[0][1] == out[1][1] == 7
    assert torch.equal(out[0][0], out[1][0]) and out[0][2] == out[1][2]


def test_capture_takes_separate_launches():
    """A V-cycle recorded into a graph runs as separate launches and gives the same result on
    every replay, with eager work in between."""
    from paper_2505_10857_amd import Solver2D, _abi as A
    s = Solver2D(wedge_problem(64, 32), device="cuda", nu1=3, nu2=3)
    J, rhs = _operator(64, 32, 9, A.NMG_FP64)
    ref = torch.zeros_like(rhs)
    s.vcycle(J, rhs, ref, setup=True)
    dU = torch.zeros_like(rhs)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        s.vcycle(None, rhs, dU, setup=False)
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=side):
        s.vcycle(None, rhs, dU, setup=False)
    for _ in range(3):
        dU.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(dU, ref)
        eager = torch.zeros_like(rhs)
        s.vcycle(None, rhs, eager, setup=False)
        assert torch.equal(eager, ref)
