"""linear.train_step / infer_step (one quantise call per tensor, biases of the
outputs in the matmul launches) against the separate calls they stand for
(fp8_scale_bias, fp8_cast_e4 / e5, the matmuls with the epilogue amax,
fp8_bias_from_amax): every code, bias, amax, flag and output, bit for bit,
on sizes whose matmuls take each kernel, with and without a margin, twice (the
workspaces are reused)."""
import pytest
import torch

import mm_routes as R
from paper_2309_17224_amd import fp8lin as F
from paper_2309_17224_amd import linear as L
from paper_2309_17224_amd import workloads as wl

pytestmark = pytest.mark.gpu


def bits(t):
    return t.view(torch.int16) if t.dtype == torch.bfloat16 else t.view(torch.int32) if t.dtype == torch.float32 else t


SIZES = [(1024, 768, 768), (255, 264, 136), (48, 512, 640), (16, 128, 384), (1, 8, 8), (1152, 2432, 2304)]


def test_routes():
    """Forward, grad-input and grad-weight products each take each kernel at
    one of the sizes."""
    for product in (lambda m, k, n: (m, n, k), lambda m, k, n: (m, k, n), lambda m, k, n: (k, n, m)):
        assert {R.kernel(*product(*s)) for s in SIZES} == {R.RAGGED, R.STREAM, R.MAIN}


@pytest.mark.parametrize("size", SIZES, ids=str)
@pytest.mark.parametrize("margin", [0, 3])
def test_step_is_the_separate_calls(gpu, size, margin):
    M, K, N = size
    b = L.alloc(M, K, N, gpu)
    for rep in range(2):
        x, w, dy = (wl.small(r, c, s, 10 * rep + r + c).to(gpu) for r, c, s in ((M, K, 1.0), (K, N, 0.02), (M, N, 1e-3)))
        L.train_step(x, w, dy, b, margin)
        ref = {}
        for name, t, fmt, mg in (("x", x, F.E4M3, 0), ("w", w, F.E4M3, 0), ("g", dy, F.E5M2, margin)):
            ref["b" + name], ref["amax_" + name], ref["flags_" + name] = F.fp8_scale_bias(t, fmt, mg)
            cast = F.fp8_cast_e4 if fmt == F.E4M3 else F.fp8_cast_e5
            codes = {"x": ("x8", "x8t"), "w": ("w8", "w8t"), "g": ("dy8", "dy8t")}[name]
            ref[codes[0]], ref[codes[1]] = cast(t, ref["b" + name], want_qT=True)
        am = torch.zeros(2, dtype=torch.int32, device=gpu)
        ref["y"] = F.fp8_linear_fwd(ref["x8"], ref["bx"], ref["w8t"], ref["bw"], y_amax_bits=am[0:1])
        ref["dx"] = F.fp8_linear_bwd_dx(ref["dy8"], ref["bg"], ref["w8"], ref["bw"], dx_amax_bits=am[1:2])
        ref["dw"] = F.fp8_linear_bwd_dw(ref["x8t"], ref["bx"], ref["dy8t"], ref["bg"])
        ref["amax_y"], ref["amax_dx"] = am[0:1], am[1:2]
        ref["by"], ref["flags_y"] = F.fp8_bias_from_amax(am[0:1], F.E4M3, 0)
        ref["bdx"], ref["flags_dx"] = F.fp8_bias_from_amax(am[1:2], F.E5M2, margin)
        torch.cuda.synchronize()
        for name, r in ref.items():
            assert torch.equal(bits(getattr(b, name)), bits(r)), name
        assert not b.bws.any()
        L.infer_step(x, b)
        torch.cuda.synchronize()
        assert torch.equal(bits(b.y), bits(ref["y"])) and torch.equal(b.x8, ref["x8"])


def test_step_refuses_strided_tensors(gpu):
    b = L.alloc(16, 32, 64, gpu)
    with pytest.raises(ValueError):
        L.infer_step(wl.small(16, 64, 1.0, 1).to(gpu)[:, :32], b)


def test_buffers_made_by_hand(gpu):
    """Buffers without the in-launch bias workspace and with one that only
    fp8_scale_bias's partials fill (4096 x 8 has fewer of them than tiles): the
    same step, and nothing allocated by it."""
    M, K, N = 4096, 8, 16
    full = L.alloc(M, K, N, gpu)
    assert F.fp8_scale_bias_ws_bytes(M * N) < F.fp8_quantise_ws_bytes(M, N)
    names = ("w8", "w8t", "x8", "x8t", "dy8", "dy8t", "y", "dx", "dw", "scal")
    own = L.LinearBuffers(M, K, N, gpu, *(torch.zeros_like(getattr(full, n)) for n in names), F.workspace(M * N, gpu))
    x, w, dy = (wl.small(r, c, s, r + c).to(gpu) for r, c, s in ((M, K, 1.0), (K, N, 0.02), (M, N, 1e-3)))
    L.train_step(x, w, dy, full)
    L.train_step(x, w, dy, own)
    torch.cuda.synchronize()
    made = torch.cuda.memory_stats()["allocation.all.allocated"]
    L.train_step(x, w, dy, own)
    L.infer_step(x, own)
    torch.cuda.synchronize()
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == made
    for n in names:
        assert torch.equal(bits(getattr(own, n)), bits(getattr(full, n))), n
