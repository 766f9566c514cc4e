"""Replayed Krylov graphs (N >= 128, one lane) against direct launches, bit for bit, where what a graph holds by value or
reads at replay changes between calls: the potential's index box (moved, smaller within the same sixteenth of the rows, in
another sixteenth), L and M (the tail's table), the batch (small ones form the Gram-Schmidt coefficients in the update's
launch; at ten entries the choice differs between these boxes), a larger grid in between.
"""
import numpy as np
import pytest

from oracle import dbar_oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1508_02363_amd import dbar as D  # noqa: E402

N = 128
# rows of the potential (whole tiles of four): 40 of them, moved, 36 (the same sixteenth), 52 (another), all
ROWS = [(40, 80), (44, 84), (44, 80), (40, 92), (0, N), (40, 80)]


def potential(L, rows):
    g = O.make_grid(N, L)
    r = np.arange(N)[:, None]
    return np.where((r >= rows[0]) & (r < rows[1]), (1.2 + 0.9j) * np.exp(-np.abs(g.z / L) ** 2), 0.0)


def both(Q, ks, L, M, **kw):
    got = D.solve(Q, ks, L, M=M, use_graph=1, **kw)
    want = D.solve(Q, ks, L, M=M, use_graph=0, **kw)
    assert [(a.iters, a.outer, a.status) for a in got[2]] == [(a.iters, a.outer, a.status) for a in want[2]], (L, M)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), (L, M)


@pytest.mark.parametrize("prec", [D.DBAR_FP64, D.DBAR_MIXED])
@pytest.mark.parametrize("method", [D.DBAR_METHOD_PLAIN, D.DBAR_METHOD_ITERATED])
@pytest.mark.parametrize("nk", [1, 3, 10, 33])
def test_replays_follow_the_box_and_the_grid(nk, method, prec):
    kw = dict(tol=1e-11, precision=prec, method=method, batch=nk, lanes=1)
    D.release()
    for turn in range(2):
        for L, M in ((2.0, 11), (2.5, 11), (2.5, 5)):
            ks = [(j % 5 - 2 + 1j * (j % 3 - 1)) / (2 * L) for j in range(nk)]
            for rows in ROWS:
                both(potential(L, rows), ks, L, M, **kw)
        D.solve(np.zeros((2 * N, 2 * N)) + 0.1 * turn, [0.5], 2.0, precision=prec, lanes=1)  # new buffers


@pytest.mark.parametrize("prec", [D.DBAR_FP64, D.DBAR_MIXED])
def test_replays_where_cycles_end_at_the_restart_length(prec):
    """Windowed cycles that stall and full ones after them, in one set of graphs."""
    g = O.make_grid(N, 4.0)
    for amp in (6.0, 1.0, 6.0):
        both(amp * (0.8 + 0.6j) * np.exp(-np.abs(g.z) ** 2), [0.5 + 0.5j, -1 + 0.3j, 2 - 1j], 4.0, 11, tol=1e-11, precision=prec,
             restart=8, lanes=1, batch=3)
