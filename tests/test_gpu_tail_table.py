"""The tail table of the x-space operator (rows' epilogue up to N = 1024): grids whose points lie in the series part, across
the closed form and beyond the radius where every P(n+1, u) is 1, one after the other through the same workspace, against
the iteration on S, which evaluates the tail at every point; N = 2048 has no table.

Tolerance: both solves stop at a relative residual of 1e-12 and the discrete systems have condition numbers below 50, so
they agree to 1e-10 of the largest value.
"""
import numpy as np
import pytest

from oracle import dbar_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1508_02363_amd import dbar as D  # noqa: E402


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("N,L,M", [(16, 0.7, 11), (64, 1.0, 15), (64, 1.0, 3), (64, 5.0, 3), (128, 4.0, 11), (512, 12.0, 15),
                                   (1024, 20.0, 11), (2048, 20.0, 11)])
def test_table_solve_matches_the_iteration_on_S(N, L, M, prec):
    g = O.make_grid(N, L)
    w = 0.2 * g.x[-1]
    Q = (0.6 - 0.3j) / w * np.exp(-np.abs(g.z - (0.3 + 0.2j) * w) ** 2 / w ** 2)
    ks = [0.4 - 0.3j, 1.1 + 0.2j]
    kw = dict(M=M, tol=1e-12, precision=D.DBAR_FP64 if prec == "fp64" else D.DBAR_MIXED)
    S, m, info = D.solve(Q, ks, L, **kw)
    assert all(i.status == 0 for i in info)
    S2, m2, _ = D.solve(Q, ks, L, space=D.DBAR_SPACE_XI, **kw)
    for j in range(len(ks)):
        assert np.max(np.abs(S[j] - S2[j])) <= 1e-10 * np.max(np.abs(S2[j]))
        assert np.max(np.abs(m[j] - m2[j])) <= 1e-10 * np.max(np.abs(m2[j]))


@pytest.mark.parametrize("N,L,M", [(8, 1.0, 15), (64, 1.0, 3), (64, 4.0, 11), (512, 12.0, 15)])
def test_single_application_with_its_own_table(N, L, M):
    """The allocation-free application makes the table in every call, whatever grid the last one had: against the oracle to
    1e-12 of the largest value, as for every operator test in FP64."""
    g = O.make_grid(N, L)
    Q = (0.5 - 0.3j) * np.exp(-np.abs(g.z - 0.3) ** 2)
    S = O.Fd(g, np.exp(-np.abs(g.z) ** 2 / 2) * (1 + 0.3j * g.z.real))
    ref = O.apply_A(g, Q, 0.4 + 0.2j, S, M)
    Qd, Sd = torch.from_numpy(Q).cuda(), torch.from_numpy(np.ascontiguousarray(S)).cuda()
    out = torch.empty_like(Sd)
    for prec in (D.DBAR_FP64, D.DBAR_FP32, D.DBAR_FP64):  # (the two precisions' tables share their place)
        D.apply_noalloc(Qd, 0.4 + 0.2j, Sd, out, L, M=M, precision=prec)
        torch.cuda.synchronize()
        if prec == D.DBAR_FP64:
            assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
