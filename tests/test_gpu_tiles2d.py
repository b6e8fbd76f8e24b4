"""2D residual and Jacobian on both sides of the rules that pick their kernels: grids of a few cells, ragged
tiles, interior and border rows in one launch or two, and the two tile sizes (65536 cells).  The residual
and sampled grid lines of the Jacobian against the oracle, to 1e-12 of the largest entry as in the other 2D
parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle.swe2d import Oracle2D  # noqa: E402
from swe_workloads import wedge_problem  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("jac", [9, 21])
@pytest.mark.parametrize("nx,ny,levels", [(5, 3, 1), (8, 6, 2), (14, 10, 2), (28, 20, 3), (56, 40, 4), (160, 96, 6),
                                          (192, 320, 7), (256, 256, 7), (192, 384, 7)])
def test_rows_on_both_sides_of_the_rules(nx, ny, levels, jac):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_10857_amd import Solver2D
    prob = wedge_problem(nx, ny, levels=levels, seed=5)
    s = Solver2D(prob, device=DEV, jac=jac)
    o = Oracle2D(prob)
    g = np.random.default_rng([nx, ny])
    U0 = prob.initial_guess()
    U0 = U0 * (1.0 + 0.02 * (g.random(U0.shape) - 0.5))
    U = s.state(U0)
    R, rn, res = s.residual(U)
    Ro, rno, reso = o.residual(U0)
    assert np.abs(R.cpu().numpy() - Ro).max() <= 1e-12 * np.abs(Ro).max()
    assert abs(res.item() - reso) <= 1e-12 * reso
    J = s.jacobian(U, R, rn)
    for j0 in sorted({0, 1, 2, 7, 8, ny // 2, ny - 3, ny - 1} & set(range(ny))):
        Jo = o.jacobian(U0, rows=(j0, j0 + 1), R=Ro, rn=rno, which=jac)
        Jt = np.ascontiguousarray(Jo[j0].transpose(1, 2, 3, 0))
        assert np.abs(J[:, :, :, j0, :].cpu().numpy() - Jt).max() <= 1e-12 * np.abs(Jt).max(), (nx, ny, jac, j0)
