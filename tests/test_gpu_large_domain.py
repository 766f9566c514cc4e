"""Domains on which the grid holds the potential in a single point (L from 1e2 to 1e20): the solution is there after a step or
two, up to rounding, on every grid size; small grids take the one-launch cycle only up to where it keeps to that.

Tolerance: the solves' own, a relative residual of 1e-12.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import dbar_workloads as W  # noqa: E402
from paper_1508_02363_amd import dbar as D  # noqa: E402


@pytest.mark.parametrize("prec,M,Ls", [(D.DBAR_FP64, 11, (1e2, 1e4, 1e8, 1e14, 1e20)), (D.DBAR_FP64, 0, (1e3, 1e28, 1e60)),
                                       (D.DBAR_MIXED, 3, (1e2, 1e5, 1e8, 1e10, 1e12))])
@pytest.mark.parametrize("N", [16, 32, 64, 128])
def test_one_point_potentials_converge(N, prec, M, Ls):
    for L in Ls:
        x = W.x_grid(N, L)
        with np.errstate(over="ignore", under="ignore"):
            Q = (0.7 + 0.35j) * np.exp(-(x[None, :] ** 2 + x[:, None] ** 2))
        S, m, info = D.solve(Q, [0.3 / L], L, M=M, precision=prec, max_iter=60)
        assert info[0].status == 0 and info[0].rel_residual <= 1e-12, (L, info[0])
        assert np.all(np.isfinite(S)) and np.all(np.isfinite(m)), L
