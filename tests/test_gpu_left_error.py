"""Calls of the library where the calling thread's earlier HIP call has failed and its error has not been read: none is
refused for it."""
import ctypes

import numpy as np
import pytest

import dbar_workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1508_02363_amd import dbar as D  # noqa: E402


@pytest.mark.parametrize("prec", [D.DBAR_FP64, D.DBAR_FP32])
def test_host_calls_after_a_failed_call_of_the_caller(prec):
    hip = ctypes.CDLL(D._lib.LIB_PATH)  # (the runtime's functions are found through the library that needs them)
    N, L = 32, 2.5  # (a grid of its own: the tail table is made anew)
    Q = W.potential_gaussian(N, L, 0.8 + 0.6j)
    calls = {"transform": lambda: D.transform(Q, L, precision=prec), "inverse": lambda: D.dbar_inverse(Q, L, precision=prec),
             "apply": lambda: D.apply(Q, 0.5 + 0.25j, Q, L, precision=prec), "solve": lambda: D.solve(Q, [0.5], L)[0]}
    Qd = torch.from_numpy(Q).cuda()
    out = torch.empty_like(Qd)
    calls["apply_noalloc"] = lambda: (D.apply_noalloc(Qd, 0.5 + 0.25j, Qd, out, L, precision=prec), None)[1]
    want = {name: call() for name, call in calls.items()}
    for name, call in calls.items():
        D.release()
        assert hip.hipSetDevice(99) != 0
        try:
            got = call()
            assert name == "apply_noalloc" or np.array_equal(got, want[name]), name
        finally:
            assert hip.hipGetLastError() != 0  # the caller's error is still its own to read
