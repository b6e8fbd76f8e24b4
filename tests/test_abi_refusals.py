"""Calls that are refused on the host, with the reason they are refused for (CPU only)."""
import ctypes

import pytest

from test_abi import _desc, _lib


@pytest.mark.parametrize("dim", [1, 2])
def test_nested_solve_names_the_bad_parameter(dim):
    """A bad parameter of one grid is that grid's error, not a workspace that is too small."""
    abi, L = _lib()
    grids = [_desc(abi, nx=64 >> g, levels=3 - g, jac=9 if dim == 2 else 3) for g in range(3)]
    for g, (d, _) in enumerate(grids):
        if dim == 2:
            d.dim, d.nx, d.ny, d.y1, d.by_gp = 2, 32 >> g, 16 >> g, 1.0, 8
    descs = (abi.nmg_desc * 3)(*[g[0] for g in grids])
    params = (abi.nmg_params * 3)(*[g[1] for g in grids])
    ws = L.nmg_nested_workspace_bytes(descs, 3, params)
    assert ws > 0
    U = (ctypes.c_void_p * 3)(256, 512, 768)
    st = (abi.nmg_stats * 3)()
    params[2].eps = 0.0
    assert L.nmg_nested_workspace_bytes(descs, 3, params) == 0
    assert L.nmg_nested_solve(descs, 3, params, ctypes.c_void_p(1024), ws, U, st, None) == abi.NMG_EINVAL
    assert b"eps" in L.nmg_last_error()
