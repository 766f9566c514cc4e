"""CPU tests of what the C ABI says about memory and defaults."""
import ctypes

import pytest

from paper_1508_02363_amd import _lib


@pytest.mark.parametrize("prec,basis,fp64,fp32", [(_lib.DBAR_MIXED, 21 * 8, 7, 2), (_lib.DBAR_FP64, 21 * 16, 6, 0)])
@pytest.mark.parametrize("N", [64, 512, 1024, 2048])
def test_request_footprint_holds_the_tail_table(N, prec, basis, fp64, fp32):
    """A request alone in its class: 21 basis vectors, the FP64 and FP32 arrays, and up to N = 1024 the quarter-plane table
    of the tail in FP64 and FP32."""
    arrays = (basis + 16 * fp64 + 8 * fp32) * N * N
    table = 24 * (N // 2 + 1) ** 2 if N <= 1024 else 0
    partials = 8 * (34 * 1024 + 67 * (N * N // 1024))  # sums over tiles and blocks of 1024 values
    got = _lib.load().dbar_request_footprint(ctypes.byref(_lib.Grid(N, 11, 5.0)), prec, 20)
    assert arrays + table + partials <= got <= arrays + table + partials + (64 << 10) + 40 * N


def test_default_opts_sets_every_field():
    """The defaults do not depend on what the caller's memory (or, for a NULL opts, the stack) held before."""
    opts = []
    for fill in (0x00, 0xff, 0x01):
        buf = (ctypes.c_uint8 * ctypes.sizeof(_lib.Opts))(*[fill] * ctypes.sizeof(_lib.Opts))
        o = _lib.Opts.from_buffer(buf)
        _lib.load().dbar_default_opts(ctypes.byref(o))
        opts.append({name: getattr(o, name) for name, _ in _lib.Opts._fields_})
    assert opts[0] == opts[1] == opts[2]
    assert opts[0]["lanes"] == 0 and opts[0]["restart"] == 0 and opts[0]["batch"] == 0
