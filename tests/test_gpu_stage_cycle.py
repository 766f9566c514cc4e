"""The cycle of one launch per stage (N >= 128) where its windowed steps give way: short restarts, a potential on which the
window stalls, entries that do and do not, and the iterated method's fused update against separate ones.

Tolerance: as for the same tests on smaller grids (whose cycles run in one launch): solves to 1e-12 agree to 1e-10.
"""
import numpy as np
import pytest

import dbar_workloads as W
from oracle import dbar_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1508_02363_amd import dbar as D  # noqa: E402

N, L = 128, 4.0
PRECISIONS = [D.DBAR_FP64, D.DBAR_MIXED]


def relerr(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


def strong():
    return 6.0 * (0.8 + 0.6j) * np.exp(-np.abs(O.make_grid(N, L).z) ** 2)


@pytest.mark.parametrize("prec", PRECISIONS)
@pytest.mark.parametrize("restart,window", [(4, 2), (4, 4), (6, 1)])
def test_short_restarts(restart, window, prec):
    Q = W.potential_gaussian_sum(N, L, seed=67)
    ks = W.k_disk(5, 2.5, seed=68)
    S0, m0, _ = D.solve(Q, ks, L, batch=5, precision=prec, orth_window=0, restart=40)
    S, m, info = D.solve(Q, ks, L, batch=5, precision=prec, orth_window=window, restart=restart)
    ref = O.solve(O.make_grid(N, L), Q, ks[0], tol=1e-13)
    assert relerr(S[0], ref.S) < 1e-10 and relerr(m[0], ref.m) < 1e-10
    for j in range(len(ks)):
        assert info[j].status == 0 and info[j].rel_residual <= 1e-12, j
        assert relerr(S[j], S0[j]) < 1e-10 and relerr(m[j], m0[j]) < 1e-10, j


@pytest.mark.parametrize("prec", PRECISIONS)
def test_a_stalled_window_gives_way(prec):
    """Restarts of 12 steps end unconverged under the window; the entries then orthogonalise fully and converge."""
    Q = strong()
    ks = np.array([0.5 + 0.5j, -1 + 0.3j, 2 - 1j])
    kw = dict(batch=3, precision=prec, restart=12)
    S0, m0, i0 = D.solve(Q, ks, L, batch=3, precision=prec, orth_window=0, restart=40)
    S, m, info = D.solve(Q, ks, L, **kw)
    ref = O.solve(O.make_grid(N, L), Q, ks[0], tol=1e-13)
    assert relerr(S[0], ref.S) < 1e-10 and relerr(m[0], ref.m) < 1e-10
    for j in range(len(ks)):
        assert info[j].iters > 12 and info[j].outer > i0[j].outer, j  # (a cycle ended at the restart length)
        assert info[j].status == 0 and info[j].rel_residual <= 1e-12, j
        assert relerr(S[j], S0[j]) < 1e-10 and relerr(m[j], m0[j]) < 1e-10, j


@pytest.mark.parametrize("prec", PRECISIONS)
@pytest.mark.parametrize("restart", [0, 12])
def test_entries_do_not_depend_on_each_other(restart, prec):
    """Some stall and orthogonalise fully inside launches where others keep the window: bit for bit as alone."""
    Q = strong()
    ks = np.array([0.5 + 0.5j, -1 + 0.3j, 2 - 1j, 0.1 - 0.2j, 7.5, -6j])
    kw = dict(precision=prec, restart=restart)
    S, m, info = D.solve(Q, ks, L, batch=len(ks), **kw)
    assert len({i.outer for i in info}) > 1 or restart == 0
    for j, k in enumerate(ks):
        S1, m1, i1 = D.solve(Q, [k], L, batch=1, **kw)
        assert (info[j].iters, info[j].outer) == (i1[0].iters, i1[0].outer), j
        assert np.array_equal(S[j], S1[0]) and np.array_equal(m[j], m1[0]), j


@pytest.mark.parametrize("prec", PRECISIONS)
def test_iterated_fused_update_against_separate_ones(prec):
    Q = W.potential_gaussian_sum(N, L, seed=73)
    ks = [0.0, (3 - 1j) / (2 * L), (-5 + 6j) / (2 * L), (9 + 2j) / (2 * L)]
    kw = dict(batch=4, precision=prec, method=D.DBAR_METHOD_ITERATED)
    S1, m1, i1 = D.solve(Q, ks, L, reorth=1, **kw)
    S2, m2, i2 = D.solve(Q, ks, L, reorth=2, **kw)
    for j in range(len(ks)):
        assert i1[j].status == 0 and i1[j].rel_residual <= 1e-12, j
        assert relerr(S1[j], S2[j]) < 1e-10 and relerr(m1[j], m2[j]) < 1e-10, j
        assert abs(i1[j].m1 - i2[j].m1) <= 1e-10 * max(abs(i2[j].m1), 1e-300), j
        if prec == D.DBAR_FP64:
            assert abs(i1[j].iters - i2[j].iters) <= 1, j
    ref = O.solve_iterated(O.make_grid(N, L), Q, ks[1], tol=1e-13)
    assert relerr(S1[1], ref.S) < 1e-10 and relerr(m1[1], ref.m) < 1e-10
