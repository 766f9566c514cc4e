"""Small batches, whose update launch forms the Gram-Schmidt coefficients itself, against large ones, which have a launch for
them: the same problem alone and among others, windowed and (after cycles that end at the restart length) not.

The reductions run in the same order either way, so the results are the same to the last bit.
"""
import numpy as np
import pytest

from oracle import dbar_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1508_02363_amd import dbar as D  # noqa: E402


@pytest.mark.parametrize("kw", [dict(), dict(restart=4), dict(orth_window=3), dict(method=D.DBAR_METHOD_ITERATED, restart=5)])
@pytest.mark.parametrize("prec", [D.DBAR_FP64, D.DBAR_MIXED])
@pytest.mark.parametrize("N,nk", [(128, 140), (256, 70), (512, 24)])
def test_one_problem_alone_and_in_a_batch(N, nk, prec, kw):
    L = 5.0
    g = O.make_grid(N, L)
    Q = (1.2 + 0.9j) * np.exp(-np.abs(g.z - 0.2) ** 2)
    ks = [(j % 11 - 5 + 1j * (j % 7 - 3)) / (2 * L) for j in range(nk)]
    S, m, info = D.solve(Q, ks, L, precision=prec, batch=nk, lanes=1, **kw)
    for j in (0, nk // 2, nk - 1):
        S1, m1, info1 = D.solve(Q, [ks[j]], L, precision=prec, **kw)
        assert info1[0].status == 0 and info[j].status == 0 and info1[0].iters == info[j].iters
        assert np.array_equal(S1[0], S[j]) and np.array_equal(m1[0], m[j])
