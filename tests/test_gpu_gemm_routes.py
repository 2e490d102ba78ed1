"""Matmuls off the 256 x 256 kernel: small outputs and ragged contractions.

Integer codes of small magnitude make every sum exact in fp32, so the product
of the integers, rounded to the output type, is the reference, bit for bit,
whatever the order of the sums; guard elements around the output, the
epilogue amax and the in-launch bias are checked too.

RAGGED (K not a multiple of 128: operand rows start at any byte address and
the last k-step is partial): both tile sizes (256 x 128 from 128 such tiles
on, 64 x 64 below), partial tiles, K below one 16-byte load, K one off a
multiple of 16 and of 128, odd N (unaligned output rows).
SMALL (K a multiple of 128, small tiles with the waves sharing k): one tile
and many, partial tiles in both directions, one to eight 16-row blocks of A,
K of less than one stage (128), of a partial last stage, of one, two and many
stages of each stage length (128, 256 and 512), several rounds of workgroups.
"""
import numpy as np
import pytest
import torch

from paper_2309_17224_amd import fp8lin as F
from parity_util import i32, np_bits, u32

pytestmark = pytest.mark.gpu

RAGGED = [(5, 7, 3), (1, 1, 1), (17, 33, 15), (64, 64, 16), (65, 63, 17), (130, 201, 127), (40, 130, 129),
          (300, 257, 1000), (2304, 4101, 255), (4100, 2050, 144), (2049, 2049, 15)]
SMALL = [(1, 1, 128), (1, 5000, 256), (16, 129, 640), (15, 22016, 384), (17, 2049, 1536), (32, 57, 512), (33, 1000, 256),
         (48, 12288, 128), (47, 4097, 896), (64, 15361, 512), (100, 4096, 1152), (101, 12290, 384), (160, 4100, 512),
         (161, 8190, 256), (256, 768, 3072), (301, 4095, 640), (300, 512, 1408), (1024, 768, 768), (513, 1030, 2048),
         (31, 57344, 128), (301, 12290, 4096), (511, 8200, 2176), (400, 8192, 4224)]
VALS = np.array([0, 1, 2, 3, -1, -2, -4], dtype=np.int64)
FMTS = {"fwd": (F.E4M3, F.E4M3), "dx": (F.E5M2, F.E4M3), "dw": (F.E4M3, F.E5M2)}
GUARD = 64


@pytest.mark.parametrize("shape", RAGGED + SMALL, ids=lambda s: "%dx%dx%d" % s)
@pytest.mark.parametrize("entry", list(FMTS))
@pytest.mark.parametrize("out_dt", [F.DT_BF16, F.DT_F32], ids=["bf16", "f32"])
def test_exact_product(orc, gpu, shape, entry, out_dt):
    M, N, K = shape
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    ia, ib = rng.integers(0, len(VALS), (M, K)), rng.integers(0, len(VALS), (N, K))
    ta, tb = (torch.from_numpy(np.array([orc.encode(f, v) for v in VALS], dtype=np.uint8)[i]).to(gpu)
              for f, i in zip(FMTS[entry], (ia, ib)))
    pa, pb = (torch.tensor([b], dtype=torch.int32, device=gpu) for b in (1, 2))
    tdt = torch.bfloat16 if out_dt == F.DT_BF16 else torch.float32
    ref = torch.from_numpy((VALS.astype(np.float64)[ia] @ VALS.astype(np.float64)[ib].T) / 8.0).to(tdt)
    buf = torch.full((M * N + 2 * GUARD,), 77.0, dtype=tdt, device=gpu)
    out = buf[GUARD:GUARD + M * N].view(M, N)
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
    assert np.array_equal(np_bits(out), np_bits(ref))
    assert bool((buf[:GUARD] == 77.0).all()) and bool((buf[-GUARD:] == 77.0).all())
