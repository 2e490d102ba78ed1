"""Quantise and cast at the edges of the 128 x 128 tiles and at any alignment.

Rows past the last whole tile and columns past the last group of eight take
clamped or shifted vector loads, and inputs, codes and transposed codes are
read and written at whatever byte address their offset and stride give.
Bar: bit for bit the oracle's amax, bias and codes; nothing written outside
the codes (guard bytes).  Shapes: rows and columns one off 8 and 128, fewer
than eight columns, one row, both sides of the size up to which one launch
does it all (160 KiB); every input also as a strided view that starts
one element into its storage.
"""
import numpy as np
import pytest
import torch

from paper_2309_17224_amd import fp8lin as F
from paper_2309_17224_amd import workloads as wl
from parity_util import i32, np_bits, u32

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (1, 5), (1, 9), (1, 129), (1, 40001), (3, 7), (5, 128), (127, 129), (128, 120), (129, 127), (136, 8), (45, 300), (301, 264), (255, 1001),
          (20, 4096), (21, 4096), (4099, 8), (9103, 9), (1025, 129), (1001, 1000), (384, 256),
          (2, 3), (4, 2), (2, 4096), (9, 260), (1000, 1), (300, 3), (1025, 4), (129, 7), (30001, 6)]


def view_of(x, strided):
    """x on the GPU, dense or as a view one element into rows 3 elements longer."""
    if not strided:
        return x.cuda()
    rows, cols = x.shape
    buf = torch.full((rows * (cols + 3) + 1,), float("inf"), dtype=x.dtype)
    v = buf[1:].view(rows, cols + 3)[:, :cols]
    v.copy_(x)
    return buf.cuda()[1:].view(rows, cols + 3)[:, :cols]


def guarded(rows, cols, pad):
    """uint8 codes [rows, cols] with row stride cols + pad, one byte into a guarded buffer."""
    buf = torch.full((rows * (cols + pad) + 2,), 0xA5, dtype=torch.uint8, device="cuda")
    return buf, buf[1:-1].view(rows, cols + pad)[:, :cols]


def guard_kept(buf, rows, cols, pad):
    b = buf.cpu().numpy()
    tail = b[1:-1].reshape(rows, cols + pad)[:, cols:]
    return b[0] == 0xA5 and b[-1] == 0xA5 and bool((tail == 0xA5).all())


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%d" % s)
@pytest.mark.parametrize("strided", [False, True], ids=["dense", "strided"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("fmt", [F.E4M3, F.E5M2])
def test_tile_edges(orc, gpu, shape, strided, dtype, fmt):
    rows, cols = shape
    x = (wl.small(rows, cols, 1.0, 7 * rows + cols).float() * 1.37).to(dtype)
    x[rows - 1, cols - 1] = -11.25              # the amax in the last corner
    xb = np_bits(x)
    ob, oa, ofl = orc.scale_bias(xb, fmt)
    oq, oqT = orc.cast(xb, fmt, ob, transpose=True)
    xd = view_of(x, strided)
    pad = 3 if strided else 0
    for pred in (None, ob, ob - 1):
        bq, q = guarded(rows, cols, pad)
        bt, qT = guarded(cols, rows, pad)
        p = None if pred is None else torch.tensor([pred], dtype=torch.int32, device=gpu)
        _, _, b, a, fl = F.fp8_quantise(xd, fmt, bias_pred=p, q=q, qT=qT)
        torch.cuda.synchronize()
        assert (i32(b), u32(a), u32(fl)) == (ob, oa, ofl), f"prediction {pred}"
        assert np.array_equal(q.cpu().numpy(), oq) and np.array_equal(qT.cpu().numpy(), oqT), f"prediction {pred}"
        assert guard_kept(bq, rows, cols, pad) and guard_kept(bt, cols, rows, pad)


@pytest.mark.parametrize("cols", [3, 8, 13, 260])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("fmt", [F.E4M3, F.E5M2, F.E4_A, F.E5_A])
def test_special_values_in_one_row(orc, gpu, cols, dtype, fmt):
    """A single row has loads of its own: zeros, infinities and NaN of both
    signs in its first and last columns, by quantise and by cast."""
    x = wl.small(1, cols, 1.0, cols).to(dtype)
    for bad in ([], [float("inf")], [float("nan"), -0.0, float("-inf")]):
        for j, v in enumerate(bad):
            x[0, (0, cols - 1, cols // 2)[j]] = v
        if len(bad) == 3:
            x[0, cols - 1] = -torch.tensor(float("nan"))
        xb = np_bits(x)
        ob, oa, ofl = orc.scale_bias(xb, fmt, 1)
        oq, oqT = orc.cast(xb, fmt, ob, transpose=True)
        q, qT, b, a, fl = F.fp8_quantise(x.to(gpu), fmt, 1, want_qT=True)
        q2, qT2 = F.fp8_cast(x.to(gpu), fmt, b, want_qT=True)
        torch.cuda.synchronize()
        assert (i32(b), u32(a), u32(fl)) == (ob, oa, ofl)
        for got, ref in ((q, oq), (q2, oq), (qT, oqT), (qT2, oqT)):
            assert np.array_equal(got.cpu().numpy(), ref)


# (1024 elements are the most that are read one by one)
@pytest.mark.parametrize("n", [1, 7, 1023, 1024, 1025, 2049, 100003])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
def test_scale_bias_unaligned(orc, gpu, n, dtype):
    x = wl.small(1, n + 1, 1.0, n).to(dtype)[0]
    x[0] = float("inf")                          # just before the tensor
    x[n] = 9.5                                   # its last element
    b, a, fl = F.fp8_scale_bias(x.cuda()[1:], F.E4M3)
    torch.cuda.synchronize()
    assert (i32(b), u32(a), u32(fl)) == orc.scale_bias(np_bits(x[1:]), F.E4M3)


@pytest.mark.parametrize("tiles", [512, 513, 2048, 2049])
@pytest.mark.parametrize("want", ["q", "qT", "both"])
def test_fp32_cast_of_many_whole_tiles(orc, gpu, tiles, want):
    """Both ways of loading whole fp32 tiles, on both sides of where the choice
    changes: the codes of 256 tiles at a time (which load one way), those of
    the first ones the oracle's."""
    rows, step = 128 * tiles, 128 * 256
    x = torch.randn(rows, 128, generator=torch.Generator(gpu).manual_seed(tiles), device=gpu)
    x[::97, 5] = float("nan")
    x[3::101, 127] = -float("inf")
    x[7::89, 64] *= 2.0 ** -20
    b = torch.tensor([6], dtype=torch.int32, device=gpu)
    for fmt in (F.E4M3, F.E5_A):
        q, qT = F.fp8_cast(x, fmt, b, want_q=want != "qT", want_qT=want != "q")
        for r in range(0, rows, step):
            part, partT = F.fp8_cast(x[r:r + step], fmt, b, want_qT=True)
            assert q is None or torch.equal(q[r:r + step], part)
            assert qT is None or torch.equal(qT[:, r:r + step], partT)
            if r == 0:
                ref, refT = orc.cast(np_bits(x[:step].cpu()), fmt, 6, transpose=True)
                assert np.array_equal(part.cpu().numpy(), ref) and np.array_equal(partT.cpu().numpy(), refT)


@pytest.mark.parametrize("n", [1, 1024, 1025, 1031, 40000])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
def test_scale_bias_finds_the_amax_anywhere(gpu, n, dtype):
    """At every offset from a 16-byte boundary, the amax in the elements before
    the first whole vector, after the last one, and inside."""
    per = 8 if dtype == torch.bfloat16 else 4
    for off in range(per + 1):
        for at in sorted({0, min(per, n - 1), n // 2, n - 1, max(n - per, 0)}):
            x = torch.zeros(n + per + 1, dtype=dtype, device=gpu)
            x[:off] = float("nan")
            x[off + n:] = float("nan")
            x[off + at] = -3.0
            _, a, _ = F.fp8_scale_bias(x[off:off + n], F.E4M3)
            assert u32(a) == 0x40400000, (off, at)


@pytest.mark.parametrize("cols", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
@pytest.mark.parametrize("fmt", [F.E4M3, F.E5_A])
def test_special_values_in_narrow_rows(orc, gpu, cols, dtype, fmt):
    """Rows of fewer than eight columns read eight elements, those of other
    rows among them: infinities and NaN beside every row, in the last rows
    (whose vectors end at the tensor's end) and past the tensor."""
    rows = 139
    for strided in (False, True):
        x = wl.small(rows, cols, 1.0, cols).to(dtype)
        for r, v in ((0, float("inf")), (1, -0.0), (60, float("nan")), (rows - 1, -float("inf")), (rows - 2, float("nan")),
                     (rows - 3, 9.0), (rows - 7, -float("nan"))):
            x[r, (r * 5) % cols] = v
        xb = np_bits(x)
        ob, oa, ofl = orc.scale_bias(xb, fmt, 1)
        oq, oqT = orc.cast(xb, fmt, 5, transpose=True)
        xd = view_of(x, strided)
        b5 = torch.tensor([5], dtype=torch.int32, device=gpu)
        q, qT = F.fp8_cast(xd, fmt, b5, want_qT=True)
        _, _, b, a, fl = F.fp8_quantise(xd, fmt, 1)
        torch.cuda.synchronize()
        assert (i32(b), u32(a), u32(fl)) == (ob, oa, ofl)
        assert np.array_equal(q.cpu().numpy(), oq) and np.array_equal(qT.cpu().numpy(), oqT)
