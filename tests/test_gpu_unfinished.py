"""Solves that end without converging return the S and m of their last iterate, not what an earlier solve left in the
workspace: a step limit inside the first FP32 cycle of a mixed solve (whose residual evaluation normally writes no
outputs), and a potential whose energy overflows, on which no step is taken.

Tolerance of the step-limit case: three FP32 steps against three FP64 ones on a system of condition number below 50;
3 x 50 x 2^-24 < 1e-5 relative, asserted at 1e-4 (an earlier solve's outputs differ by order 1).
"""
import numpy as np
import pytest

import dbar_workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1508_02363_amd import dbar as D  # noqa: E402

L = 3.0


def relerr(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("method", [D.DBAR_METHOD_PLAIN, D.DBAR_METHOD_ITERATED])
@pytest.mark.parametrize("N", [8, 64, 128])
def test_step_limit_inside_the_first_mixed_cycle(N, method):
    other = W.potential_gaussian_sum(N, L, seed=5)
    Q = W.potential_gaussian(N, L, 0.8 + 0.6j)
    ks = [0.5, -1.0 + 0.5j]
    D.solve(other, ks, L, precision=D.DBAR_MIXED, method=method)
    S, m, info = D.solve(Q, ks, L, precision=D.DBAR_MIXED, method=method, max_iter=3)
    S2, m2, info2 = D.solve(Q, ks, L, method=method, max_iter=3)
    for j in range(len(ks)):
        assert info[j].status == D.DBAR_ENOCONV and info[j].iters == 3
        assert relerr(S[j], S2[j]) <= 1e-4 and relerr(m[j], m2[j]) <= 1e-4, (info[j], info2[j])
        assert abs(info[j].m1 - info2[j].m1) <= 1e-4 * abs(info2[j].m1)


@pytest.mark.parametrize("prec", [D.DBAR_FP64, D.DBAR_MIXED])
@pytest.mark.parametrize("method", [D.DBAR_METHOD_PLAIN, D.DBAR_METHOD_ITERATED])
@pytest.mark.parametrize("N", [16, 64])
def test_a_potential_whose_energy_overflows_leaves_zero(N, method, prec):
    """|Q|^2 overflows: the residual is not finite from the start, no step is taken and x stays 0 (S = m = 0)."""
    Q = W.potential_gaussian(N, L, 0.8 + 0.6j)
    D.solve(Q, [0.5], L, precision=prec, method=method)
    S, m, info = D.solve(1e200 * Q, [0.5], L, precision=prec, method=method)
    assert not info[0].rel_residual <= 1e-12 and info[0].iters == 0
    assert np.all(S == 0) and np.all(m == 0) and info[0].m1 == 0


def test_a_served_request_whose_energy_overflows_leaves_zero():
    """The same in a serving session, whose slot another request has used before."""
    Q = W.potential_gaussian(64, L, 0.8 + 0.6j)
    with D.Session(max_slots=1) as s:
        for q, zero in ((Q, False), (1e200 * Q, True)):
            S, m, info, _ = s.wait(s.submit(q, 0.5, L, tol=1e-12))
            assert np.any(S != 0) != zero and np.any(m != 0) != zero, info


@pytest.mark.parametrize("prec", [D.DBAR_FP64, D.DBAR_MIXED])
@pytest.mark.parametrize("N", [64, 128])
def test_an_infinite_residual_is_not_converged(N, prec):
    """||b|| overflows, so that ||r|| <= tol ||b|| holds as inf <= inf: the status says that the solve did not converge."""
    Q = W.potential_gaussian(N, L, 0.8 + 0.6j)
    _, _, info = D.solve(1e200 * Q, [0.5, 0.0], L, precision=prec, max_iter=40)
    assert all(i.status == D.DBAR_ENOCONV and i.iters == 0 for i in info), info
