"""Line kernels at the grid sizes where their shapes change (elements per thread, lines per tile, the thread limit of wide
column tiles), for every column-tile variant: the operator against the oracle and the boxed solve against variant 0.

Tolerances as for the other operator tests: 1e-12 (FP64) and 2e-5 (FP32) of the largest value; solves stop at 1e-12, so
two of them agree to 1e-11.
"""
import numpy as np
import pytest

from oracle import dbar_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1508_02363_amd import dbar as D  # noqa: E402


def relerr(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("M", [3, 11, 15])
@pytest.mark.parametrize("N", [8, 16, 32, 128, 512])
def test_every_variant(N, M):
    L = max(1.0, N / 40.0)
    g = O.make_grid(N, L)
    Q = (0.5 - 0.3j) * np.exp(-np.abs(g.z - 0.3) ** 2)
    S = O.Fd(g, np.exp(-np.abs(g.z) ** 2 / 2) * (1 + 0.3j * g.z.real))
    k = 0.4 + 0.2j
    ref = O.apply_A(g, Q, k, S, M)
    try:
        base = None
        for v in range(max(D.get_tile(N, p)[2] for p in (D.DBAR_FP64, D.DBAR_FP32))):
            for prec, tol in ((D.DBAR_FP64, 1e-12), (D.DBAR_FP32, 2e-5)):
                D.set_tile(N, prec, min(v, D.get_tile(N, prec)[2] - 1))
                assert relerr(D.apply(Q, k, S, L, M=M, precision=prec), ref) < tol, (v, prec)
            Sv, mv, info = D.solve(Q, [k, -0.5j], L, M=M, precision=D.DBAR_MIXED)
            assert all(i.status == 0 for i in info)
            if base is None:
                base = (Sv, mv)
            for j in range(2):
                assert relerr(Sv[j], base[0][j]) < 1e-11 and relerr(mv[j], base[1][j]) < 1e-11, v
    finally:
        for prec in (D.DBAR_FP64, D.DBAR_FP32):
            D.set_tile(N, prec, 0)
