"""Which kernel a matmul takes, and matmuls through a given kernel and tile:
entry points of the built library that its header does not declare, so that
the tests can state, and choose, the kernel they run."""
from __future__ import annotations

import ctypes
import os

from paper_2309_17224_amd import fp8lin as F

RAGGED, STREAM, MAIN = 0, 1, 2  # K not a multiple of 128; small tiles; 256 x 256 tiles
_i32, _i64, _vp = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p


def _lib():
    if not os.path.exists(F.LIB_PATH):
        from paper_2309_17224_amd import build
        build.build()
    L = F.lib()
    L.fp8lin_mm_route.argtypes = [_i64, _i64, _i64, _i32, _vp, _vp]
    L.fp8lin_mm_tile.argtypes = [_i32, _vp, _vp]
    L.fp8lin_mm_forced.argtypes = [_i32, _i32, _i32, _vp, _i32, _vp, _vp, _i32, _vp, _vp, _i32, _i64, _i64, _i64, _i32,
                                   _i32, _vp, _vp, _vp, _vp, ctypes.c_size_t, _vp]
    return L


def route(M: int, N: int, K: int, with_amax: bool = False):
    """(kernel, mb, nb): tiles of 16 mb x 16 nb outputs for STREAM, else zeros.
    with_amax: of a call that takes the amax or the bias of its output."""
    mb, nb = _i32(), _i32()
    kernel = _lib().fp8lin_mm_route(M, N, K, int(with_amax), ctypes.byref(mb), ctypes.byref(nb))
    return kernel, mb.value, nb.value


def kernel(M: int, N: int, K: int) -> int:
    return route(M, N, K)[0]


def stage(mb: int, nb: int) -> int:
    """Bytes of k per stage of a small tile: tiles of one stage length sum in
    one order, and 128 in that of the 256 x 256 kernel."""
    return 512 if mb + nb <= 6 else 256 if mb + nb <= 12 else 128


def workgroups(M: int, N: int, mb: int, nb: int) -> int:
    return -(-M // (16 * mb)) * -(-N // (16 * nb))


def tiles():
    """The tiles (mb, nb) the small-tile kernel is built for."""
    out, mb, nb = [], _i32(), _i32()
    while _lib().fp8lin_mm_tile(len(out), ctypes.byref(mb), ctypes.byref(nb)):
        out.append((mb.value, nb.value))
    return out


def forced(kernel, tile, a, fa, ba, b, fb, bb, out, fmt=F.E4M3, margin=0, bias=None, amax=None, flags=None, ws=None):
    """out [M, N] = 2^-(ba + bb) a [M, K] . b [N, K]^T through kernel and tile;
    with ws, the bias of out as fp8_linear_fwd_bias takes it.  Returns the status."""
    p = lambda t: None if t is None else t.data_ptr()
    M, K = a.shape
    return _lib().fp8lin_mm_forced(kernel, *tile, p(a), fa, p(ba), p(b), fb, p(bb), p(out), F._dt(out), M, b.shape[0], K,
                                   fmt, margin, p(bias), p(amax), p(flags), p(ws), 0 if ws is None else 4 * ws.numel(),
                                   F._stream())
