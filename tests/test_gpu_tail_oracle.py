"""The tail table against the oracle: one application reads it in its column tail, a solve in its row tail; neither side of
a comparison within the library is independent of it (the iteration on S reads the same table).

Tolerances: 1e-12 of the largest value for an FP64 application, as for every operator test.  A solve stops at a residual of
1e-12 of its own operator; the oracle's operator agrees with it to 1e-12 of the largest value at every point, and 2-norms
over a grid differ from largest values by less than a factor of 100 for these right-hand sides: 1e-10.  An FP32
application: 2e-5 as elsewhere; at M = 15 and |z| up to 53 the deepest moments carry the FP32 rounding (3.4e-5 on average
and 1.3e-4 at most over 24 draws with the tail's series in place of its table): 5e-4.
"""
import numpy as np
import pytest

from oracle import dbar_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1508_02363_amd import dbar as D  # noqa: E402

GRIDS = [(16, 0.7, 11), (64, 1.0, 15), (64, 1.0, 3), (64, 5.0, 3), (128, 4.0, 11), (512, 12.0, 15), (1024, 20.0, 11),
         (2048, 20.0, 11)]


def relerr(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("N,L,M", GRIDS)
def test_application_and_solve_against_the_oracle(N, L, M):
    g = O.make_grid(N, L)
    w = 0.2 * g.x[-1]
    Q = (0.6 - 0.3j) / w * np.exp(-np.abs(g.z - (0.3 + 0.2j) * w) ** 2 / w ** 2)
    S = O.Fd(g, np.exp(-np.abs(g.z / w) ** 2) * (1 + 0.3j * g.z.real / w))
    k = 0.4 - 0.3j
    om = O.omega_table(g, M)
    ref = O.apply_A(g, Q, k, S, M, om=om)
    assert relerr(D.apply(Q, k, S, L, M=M), ref) <= 1e-12
    b = O.rhs(g, Q, k)
    for prec in (D.DBAR_FP64, D.DBAR_MIXED):
        Sx, _, info = D.solve(Q, [k], L, M=M, tol=1e-12, precision=prec)
        r = b - O.apply_A(g, Q, k, Sx[0], M, om=om)
        assert info[0].status == 0 and np.linalg.norm(r) <= 1e-10 * np.linalg.norm(b), (prec, info[0])


@pytest.mark.parametrize("N,L,M,tol", [(8, 1.0, 15, 2e-5), (64, 4.0, 11, 2e-5), (512, 12.0, 11, 2e-5), (512, 12.0, 15, 5e-4)])
def test_fp32_application_against_the_oracle(N, L, M, tol):
    g = O.make_grid(N, L)
    om = O.omega_table(g, M)
    for seed in range(4):
        rng = np.random.default_rng(seed)
        c = rng.uniform(-0.5, 0.5, 4)
        Q = (0.5 - 0.3j) * np.exp(-np.abs(g.z - c[0] - 1j * c[1]) ** 2)
        S = O.Fd(g, np.exp(-np.abs(g.z - c[2]) ** 2 / 2) * (1 + 1j * c[3] * g.z.real))
        ref = O.apply_A(g, Q, 0.4 + 0.2j, S, M, om=om)
        Qd, Sd = torch.from_numpy(Q).cuda(), torch.from_numpy(np.ascontiguousarray(S)).cuda()
        out = torch.empty_like(Sd)
        D.apply_noalloc(Qd, 0.4 + 0.2j, Sd, out, L, M=M, precision=D.DBAR_FP32)
        assert relerr(out.cpu().numpy(), ref) <= tol, seed
        assert relerr(D.apply(Q, 0.4 + 0.2j, S, L, M=M, precision=D.DBAR_FP32), ref) <= tol, seed
