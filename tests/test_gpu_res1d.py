"""res of one 1D residual call: one workgroup takes all tiles of a small grid and writes res itself, a
larger grid's res is summed by a second launch.  Sizes on both sides of the tile edges and of that rule.
Both sums add at most 1280 positive terms in chains of at most 5 and trees of 8 levels, the reference in
trees, so they agree within 32 roundings."""
import dataclasses

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from swe_workloads import config2  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("n,levels", [(4, 1), (255, 1), (256, 1), (258, 2), (512, 2), (516, 3), (768, 3),
                                      (1020, 3), (1024, 3), (1032, 4), (1280, 4)])
def test_res_is_the_mean_of_the_norms(n, levels):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_10857_amd import Solver1D
    prob = dataclasses.replace(config2(0, "sub", n=2048, levels=4), n=n, levels=levels)
    s = Solver1D(prob, device=DEV)
    R, rn, res = s.residual(s.state())
    assert torch.equal(rn, R[0].abs() + R[1].abs())
    assert abs(res.item() - rn.sum().item() / n) <= 32 * 2.3e-16 * res.item()
