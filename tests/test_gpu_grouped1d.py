"""The 1D V-cycle of a small batch takes several levels a launch (tiles with margins) and starts the
bottom kernel at a smaller level; with other options every level has its own launch.  Both do the same
operations in the same order, so the states after some Newton steps are equal bit for bit.  The sizes
put 1, 2, 4 and 6 levels above the bottom, one and many tiles, ragged last tiles and grids of a few
pairs; smoothing counts widen and narrow the margins."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from swe_workloads import config2  # noqa: E402

DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


CASES = [(57 << 5, 6), (33 << 6, 7), (4096, 5), (81 << 6, 7), (12800, 8), (37 << 8, 9), (40 << 10, 11)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("jac,nu1,nu2", [(3, 2, 2), (5, 2, 2), (3, 1, 3), (3, 4, 4), (3, 0, 2), (3, 8, 8), (3, 8, 1)])
def test_grouped_levels_equal_a_launch_per_level(jac, nu1, nu2, prec):
    from paper_2505_10857_amd import BatchSolver1D
    probs = []
    for n, levels in CASES:
        p = config2(0, "sub", n=n, levels=levels)
        probs.append(dataclasses.replace(p, params=dataclasses.replace(p.params, nu1=nu1, nu2=nu2, n_max=3)))
    for group in [[p] for p in probs] + [probs]:
        out = []
        for options in (None, {"bottom_cells": 2048, "split_finest": 1}, {"bottom_cells": 512}):
            s = BatchSolver1D(group, device=DEV, precision=prec, jac=jac)
            if options:
                s.set_options(**options)
            U = s.states()
            s.solve(U)
            out.append([u.cpu().numpy() for u in U])
        for k, a in enumerate(out[0]):
            assert np.isfinite(a).all()
            assert np.array_equal(a, out[1][k]) and np.array_equal(a, out[2][k]), (group[k].n, jac, nu1, nu2, prec)
