"""Every matmul kernel and tile, on exact products.

Integer codes of small magnitude make every sum exact in fp32, so the product
of the integers, rounded to the output type, is the reference, bit for bit,
whatever the order of the sums; guard elements around the output, the
epilogue amax and the in-launch bias are checked too.

Through the entry points, each shape stating the kernel it takes:
RAGGED (K not a multiple of 128: operand rows start at any byte address and
the last k-step is partial): both tile sizes (256 x 128 from 128 such tiles
on, 64 x 64 below), partial tiles, K below one 16-byte load, K one off a
multiple of 16 and of 128, odd N (unaligned output rows).
SMALL (small tiles) and MAIN (256 x 256 tiles), as the sizes route them.

Through a given kernel: every tile the small-tile kernel is built for, with
one partial tile alone and several, partial in both directions, over K of one
128-byte step, of less than one stage, of a partial last stage, of two, three
and many stages of each stage length (128, 256, 512); and the 256 x 256 kernel
with no, 64, 128 and 192 columns wide tiles in its last round, over K of one,
two, three and more steps.
"""
import numpy as np
import pytest
import torch

import mm_routes as R
from paper_2309_17224_amd import fp8lin as F
from parity_util import i32, np_bits, u32

pytestmark = pytest.mark.gpu

RAGGED = [(5, 7, 3), (1, 1, 1), (17, 33, 15), (64, 64, 16), (65, 63, 17), (130, 201, 127), (40, 130, 129),
          (300, 257, 1000), (2304, 4101, 255), (4100, 2050, 144), (2049, 2049, 15)]
SMALL = [(1, 1, 128), (1, 5000, 256), (16, 129, 640), (15, 22016, 384), (17, 2049, 1536), (32, 57, 512), (33, 1000, 256),
         (47, 4097, 896), (64, 15361, 512), (100, 4096, 1152), (160, 4100, 512), (256, 768, 3072), (301, 4095, 640),
         (300, 512, 1408), (1024, 768, 768), (513, 1030, 2048), (31, 57344, 128), (513, 4100, 5248)]
MAIN = [(101, 12290, 384), (161, 8190, 256), (301, 12290, 4096), (511, 8200, 2176), (700, 4099, 128), (1030, 2305, 256),
        (400, 8192, 4224)]
SHAPES = [(R.RAGGED, s) for s in RAGGED] + [(R.STREAM, s) for s in SMALL] + [(R.MAIN, s) for s in MAIN]
VALS = np.array([0, 1, 2, 3, -1, -2, -4], dtype=np.int64)
FMTS = {"fwd": (F.E4M3, F.E4M3), "dx": (F.E5M2, F.E4M3), "dw": (F.E4M3, F.E5M2)}
GUARD = 64


def operands(orc, gpu, entry, M, N, K):
    """Codes of the two operands, their biases, and the product / 8 in fp32."""
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    ia, ib = rng.integers(0, len(VALS), (M, K)), rng.integers(0, len(VALS), (N, K))
    ta, tb = (torch.from_numpy(np.array([orc.encode(f, v) for v in VALS], dtype=np.uint8)[i]).to(gpu)
              for f, i in zip(FMTS[entry], (ia, ib)))
    pa, pb = (torch.tensor([b], dtype=torch.int32, device=gpu) for b in (1, 2))
    va, vb = (torch.from_numpy(VALS.astype(np.float32)[i]) for i in (ia, ib))
    return ta, pa, tb, pb, (va @ vb.t()) / 8.0  # |sums| < 2^24: exact


def guarded(gpu, M, N, dt):
    buf = torch.full((M * N + 2 * GUARD,), 77.0, dtype=dt, device=gpu)
    return buf, buf[GUARD:GUARD + M * N].view(M, N)


def guards_kept(buf):
    return bool((buf[:GUARD] == 77.0).all()) and bool((buf[-GUARD:] == 77.0).all())


@pytest.mark.parametrize("kernel,shape", SHAPES, ids=lambda s: "%dx%dx%d" % s if isinstance(s, tuple) else str(s))
@pytest.mark.parametrize("entry", list(FMTS))
@pytest.mark.parametrize("out_dt", [F.DT_BF16, F.DT_F32], ids=["bf16", "f32"])
def test_exact_product(orc, gpu, kernel, shape, entry, out_dt):
    M, N, K = shape
    assert R.kernel(M, N, K) == kernel
    ta, pa, tb, pb, prod = operands(orc, gpu, entry, M, N, K)
    tdt = torch.bfloat16 if out_dt == F.DT_BF16 else torch.float32
    ref = prod.to(tdt)
    buf, out = guarded(gpu, M, N, tdt)
    if entry == "dw":
        F.fp8_linear_bwd_dw(ta, pa, tb, pb, dw=out)
        torch.cuda.synchronize()
    else:
        fn, kw = (F.fp8_linear_fwd, {"y": out}) if entry == "fwd" else (F.fp8_linear_bwd_dx, {"dx": out})
        am = torch.full((1,), 0x7FFFFFFF, dtype=torch.int32, device=gpu)
        fn(ta, pa, tb, pb, **kw, **{("y" if entry == "fwd" else "dx") + "_amax_bits": am})
        fb = F.fp8_linear_fwd_bias if entry == "fwd" else F.fp8_linear_bwd_dx_bias
        ws = F.bias_workspace(gpu)
        y2, b, a, fl = fb(ta, pa, tb, pb, F.E4M3, 1, out_dt=out_dt, ws=ws)
        torch.cuda.synchronize()
        assert np.array_equal(np_bits(y2), np_bits(ref)) and not ws.any()
        ob, oa, ofl = orc.scale_bias(np_bits(ref), F.E4M3, 1)
        assert (i32(b), u32(a), u32(fl)) == (ob, oa, ofl) and u32(am) == oa
    assert np.array_equal(np_bits(out), np_bits(ref)) and guards_kept(buf)


def check_forced(orc, gpu, kernel, tile, shape, entry, tdt):
    M, N, K = shape
    ta, pa, tb, pb, prod = operands(orc, gpu, entry, M, N, K)
    ref = prod.to(tdt)
    oa = orc.scale_bias(np_bits(ref), F.E4M3, 1)
    for mode in ("plain", "amax", "bias"):
        buf, out = guarded(gpu, M, N, tdt)
        z = torch.full((3,), 0x7FFFFFF, dtype=torch.int32, device=gpu)
        ws = F.bias_workspace(gpu)
        kw = {"plain": {}, "amax": {"amax": z[1:2]}, "bias": dict(bias=z[0:1], amax=z[1:2], flags=z[2:3], ws=ws)}[mode]
        assert R.forced(kernel, tile, ta, FMTS[entry][0], pa, tb, FMTS[entry][1], pb, out, F.E4M3, 1, **kw) == F.OK
        torch.cuda.synchronize()
        where = f"{tile} {shape} {entry} {mode}"
        assert np.array_equal(np_bits(out), np_bits(ref)) and guards_kept(buf), where
        if mode != "plain":
            assert u32(z[1]) == oa[1], where
        if mode == "bias":
            assert (i32(z[0]), u32(z[2])) == (oa[0], oa[2]) and not ws.any(), where


@pytest.mark.parametrize("tile", R.tiles(), ids=lambda t: "%dx%d" % t)
def test_every_small_tile(orc, gpu, tile):
    mb, nb = tile
    entries = list(FMTS)
    for i, K in enumerate((128, 256, 384, 512, 640, 1152, 2176)):
        # two tile rows, the second of one row or all but one; three tile
        # columns, the last partial with N odd, or whole
        M = 16 * mb + (1 if i % 2 else 16 * mb - 1)
        N = 2 * 16 * nb + (16 * nb if i % 3 == 2 else 16 * nb // 2 + 3)
        for tdt in (torch.bfloat16, torch.float32):
            check_forced(orc, gpu, R.STREAM, tile, (M, N, K), entries[i % 3], tdt)
    check_forced(orc, gpu, R.STREAM, tile, (max(1, 16 * mb - 9), 5, 896), "fwd", torch.bfloat16)  # one partial tile alone
    check_forced(orc, gpu, R.STREAM, tile, (1, 16 * nb, 128), "dx", torch.float32)


# (M, N): the 256 x 256 kernel with all its columns in tiles 64, 128 and 192
# wide, whole rounds and then 192 or 64 wide ones, and none narrower.
MAIN_GRIDS = [(255, 300), (700, 1027), (300, 8203), (515, 8205), (257, 16390), (4000, 11001), (4000, 8300), (4097, 8190)]


@pytest.mark.parametrize("grid", MAIN_GRIDS, ids=lambda g: "%dx%d" % g)
def test_main_kernel(orc, gpu, grid):
    M, N = grid
    steps = (1, 2, 3, 6) if M * N < 10 ** 7 else (1, 3)
    for i, nk in enumerate(steps):
        check_forced(orc, gpu, R.MAIN, (0, 0), (M, N, 128 * nk), list(FMTS)[i % 3], (torch.bfloat16, torch.float32)[i % 2])


def test_forced_rejects(gpu):
    t = torch.zeros((16, 256), dtype=torch.uint8, device=gpu)
    z = torch.zeros(1, dtype=torch.int32, device=gpu)
    out = torch.zeros((16, 16), dtype=torch.float32, device=gpu)
    args = (t, F.E4M3, z, t, F.E4M3, z, out)
    assert R.forced(R.STREAM, (7, 7), *args) == F.EINVAL       # no such tile
    assert R.forced(3, (0, 0), *args) == F.EINVAL              # no such kernel
    odd = t[:, :100].contiguous()
    assert R.forced(R.MAIN, (0, 0), odd, F.E4M3, z, odd, F.E4M3, z, out) == F.EINVAL  # K not a multiple of 128


@pytest.mark.parametrize("K", [*range(1, 16), 48, 112, 240])
def test_contraction_of_few_or_whole_loads(orc, gpu, K):
    """K < 16: a row's bytes come in one to three overlapping loads; K a
    multiple of 16: in whole ones, none past the last."""
    M, N = 67, 130
    ta, pa, tb, pb, prod = operands(orc, gpu, "fwd", M, N, K)
    assert R.kernel(M, N, K) == R.RAGGED
    y = F.fp8_linear_fwd(ta, pa, tb, pb, out_dt=F.DT_F32)
    torch.cuda.synchronize()
    assert np.array_equal(np_bits(y), np_bits(prod))
