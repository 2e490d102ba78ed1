"""Workloads over which the speed of the FP8 path is followed.

Each case is one pass of a user's program through the public entry points:
a training step of one linear layer (forward and backward with the quantise of
its weight, input and gradient), the four linears of a Llama 2 decoder layer
with post-training-quantised weights at any number of tokens (token-by-token
decode, batched decode, short and long prefill), a whole decoder layer, its
attention alone, and the quantisation of a checkpoint's weights.  Sizes are
those of the configurations in paper_2309_17224_amd/workloads.py, with token
counts as they come in use: one token, a batch of sequences, odd lengths.

listed() holds the cases that are always followed, draw() gives more of the
same ranges.  prepare() makes the inputs on the GPU from a seed, run() does one
pass, exact() computes its floating outputs in fp64 with plain torch.
"""
import math

import torch

from paper_2309_17224_amd import decoder as D
from paper_2309_17224_amd import fp8lin as F
from paper_2309_17224_amd import linear as L
from paper_2309_17224_amd import workloads as wl

# Llama 2 decoder dimensions by layer configuration: d_model, heads, key-value
# heads, ffn, weight standard deviation (head dimension 128).
MODELS = {"7b": (4096, 32, 32, 11008, 0.02), "70b": (8192, 64, 8, 28672, 0.01), "tiny": (512, 8, 2, 1408, 0.05)}


def listed():
    return [
        # The smallest linear that is trained (GPT 111M, 1024 tokens), call by
        # call: launches and host work count.
        {"name": "train-111m-calls", "kind": "train", "m": 1024, "k": 768, "n": 768, "quant": "calls", "dist": "normal"},
        # An ordinary training step (Llama 2 7B up projection), one graph per
        # step, biases predicted from the step before; outlier channels.
        {"name": "train-7b-up", "kind": "train", "m": 4096, "k": 4096, "n": 11008, "quant": "predicted", "dist": "outlier"},
        # The largest: Llama 2 13B fused QKV, 8192 tokens, gradient rows over
        # ten binades.
        {"name": "train-13b-qkv", "kind": "train", "m": 8192, "k": 5120, "n": 15360, "quant": "predicted", "dist": "rows"},
        # A micro-batch of an odd number of tokens (unpadded sequences), delayed
        # scaling: the grad-weight product contracts over the tokens.
        {"name": "train-7b-odd-delayed", "kind": "train", "m": 1531, "k": 4096, "n": 4096, "quant": "delayed", "dist": "normal"},
        # Token-by-token decode of one sequence.
        {"name": "serve-7b-1", "kind": "serve", "model": "7b", "m": 1},
        # Decode of 16 sequences through the 70B linears: the weights stream
        # from memory.
        {"name": "serve-70b-16", "kind": "serve", "model": "70b", "m": 16},
        # Batched decode of more sequences than one matrix tile holds.
        {"name": "serve-7b-48", "kind": "serve", "model": "7b", "m": 48},
        # A short prompt of odd length.
        {"name": "serve-7b-301", "kind": "serve", "model": "7b", "m": 301},
        # Prefill of a whole decoder layer, the largest model: all four linears
        # and everything between them.
        {"name": "layer-70b-2048", "kind": "layer", "model": "70b", "rows": 2048, "seq": 2048, "per": "tensor"},
        # The same for a batch of three shorter prompts with one activation
        # bias per sequence.
        {"name": "layer-7b-3x717-seq", "kind": "layer", "model": "7b", "rows": 2151, "seq": 717, "per": "sequence"},
        # Causal attention without head grouping over two odd-length sequences,
        # with the quantise of its output.
        {"name": "attention-7b-2x1999", "kind": "attention", "model": "7b", "rows": 3998, "seq": 1999},
        # Checkpoint load: one fp32 weight to codes and transposed codes.
        {"name": "ptq-fp32-70b-qkv", "kind": "ptq", "k": 8192, "n": 10240, "dtype": "f32"},
    ]


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "serve", "serve", "serve", "serve", "layer", "attention", "ptq"])
    if kind == "train":
        widths = [768, 3072, 4096, 5120, 8192, 11008, 15360]
        m = _logint(rng, 64, 8192)
        if rng.random() < 0.5:
            m = -(-m // 128) * 128       # padded batches are as common as odd ones
        k, n = rng.choice(widths), rng.choice(widths)
        if rng.random() < 0.2:           # layers of other widths
            k, n = 8 * _logint(rng, 24, 1024), 8 * _logint(rng, 24, 1024)
        while m * k * n > 8192 * 5120 * 15360:
            m = max(64, m // 2)
        return {"kind": "train", "m": m, "k": k, "n": n, "quant": rng.choice(["calls", "predicted", "predicted", "twopass", "delayed"]),
                "dist": rng.choice(["normal", "outlier", "rows"])}
    if kind == "serve":
        return {"kind": "serve", "model": rng.choice(["7b", "7b", "70b"]), "m": _logint(rng, 1, 2048)}
    if kind == "layer":
        model = rng.choice(["tiny", "7b", "7b", "70b"])
        seq = _logint(rng, 64, 2048)
        rows = min(3072, seq * rng.randint(1, 4)) if model != "70b" else min(2048, seq * rng.randint(1, 2))
        return {"kind": "layer", "model": model, "rows": rows, "seq": seq, "per": rng.choice(["tensor", "sequence"])}
    if kind == "attention":
        seq = _logint(rng, 128, 4096)
        return {"kind": "attention", "model": rng.choice(["7b", "70b"]), "rows": min(4096, seq * rng.randint(1, 4)), "seq": seq}
    return {"kind": "ptq", "k": 8 * _logint(rng, 96, 1280), "n": 8 * _logint(rng, 96, 1280), "dtype": rng.choice(["f32", "bf16"])}


# ------------------------------------------------------------------ inputs
def _randn(gen, rows, cols, std=1.0, dtype=torch.bfloat16):
    x = torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float32)
    return x.mul_(std).to(dtype)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _train_inputs(case, seed):
    g, m, k, n = _gen(seed), case["m"], case["k"], case["n"]
    x, w, dy = _randn(g, m, k), _randn(g, k, n, 0.02), _randn(g, m, n, 1e-4)
    if case["dist"] == "outlier":        # 0.1 % of the channels 50 times as large
        idx = torch.randperm(k, generator=g, device="cuda")[:max(1, round(0.001 * k))]
        x[:, idx] *= 50
    elif case["dist"] == "rows":         # gradient rows spread over ten binades
        u = torch.rand((m, 1), generator=g, device="cuda") * 10 - 7
        dy = (dy.float() * torch.exp2(u)).to(torch.bfloat16)
    return x, w, dy


def _linears(case):
    d, nh, nkv, ffn, std = MODELS[case["model"]]
    return [("qkv", d, (nh + 2 * nkv) * 128, std), ("o", nh * 128, d, std), ("gateup", d, 2 * ffn, std), ("down", ffn, d, std)]


def _serve_inputs(case, seed):
    g, t = _gen(seed), {}
    for name, k, n, std in _linears(case):
        t["W" + name] = _randn(g, k, n, std)
        t["X" + name] = _randn(g, case["m"], k)
    return t


def _layer_inputs(case, seed):
    g = _gen(seed)
    d, nh, nkv, ffn, std = MODELS[case["model"]]
    w = {"g_attn": _randn(g, 1, d, 0.1).add_(1.0), "g_mlp": _randn(g, 1, d, 0.1).add_(1.0)}
    for key, (_, k, n, s) in zip(("Wqkv", "Wo", "Wgu", "Wd"), _linears(case)):
        w[key] = _randn(g, k, n, s)
    return w, _randn(g, case["rows"], d)


def _attention_inputs(case, seed):
    _, nh, nkv, _, _ = MODELS[case["model"]]
    return _randn(_gen(seed), case["rows"], (nh + 2 * nkv) * 128)


# ------------------------------------------------------------------ prepare / run
def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        x, w, dy = _train_inputs(case, seed)
        m, k, n = case["m"], case["k"], case["n"]
        if case["quant"] == "calls":
            return {"kind": "calls", "x": x, "w": w, "dy": dy, "b": L.alloc(m, k, n, "cuda")}
        load = wl.Workload("train", 0, "one linear", (wl.Tensor("X", m, k, "normal"), wl.Tensor("W", k, n, "normal"),
                                                      wl.Tensor("dY", m, n, "normal")),
                           (wl.Linear("linear", "X", "W", "dY", m, k, n),))
        step = L.WorkloadStep(load, {"X": x, "W": w, "dY": dy}, "cuda", quant=case["quant"])
        step.run()                       # the step before: its biases are the predictions
        step.capture()
        return {"kind": "step", "step": step}
    if kind == "serve":
        t = _serve_inputs(case, seed)
        load = wl.Workload("serve", 0, "the linears of a decoder layer", (),
                           tuple(wl.Linear(name, "X" + name, "W" + name, None, case["m"], k, n) for name, k, n, _ in _linears(case)),
                           train=False)
        step = L.WorkloadStep(load, t, "cuda")
        step.prepare_inference()
        step.run()
        step.capture()
        return {"kind": "step", "step": step}
    if kind == "layer":
        w, h = _layer_inputs(case, seed)
        d, nh, nkv, ffn, std = MODELS[case["model"]]
        cfg = wl.LayerConfig("layer", 0, "a decoder layer", d, nh, nkv, 128, ffn, case["rows"], case["seq"], std)
        layer = D.DecoderLayer(cfg, w, "cuda", bias_per=case["per"])
        layer.H.copy_(h)
        layer.run()
        layer.capture()
        return {"kind": "layer", "layer": layer}
    if kind == "attention":
        qkv = _attention_inputs(case, seed)
        _, nh, nkv, _, _ = MODELS[case["model"]]
        rows = case["rows"]
        scal = torch.zeros(3, dtype=torch.int32, device="cuda")
        ws = torch.empty(F.llama_attention_ws_bytes(rows, case["seq"], nh), dtype=torch.uint8, device="cuda")
        q = torch.empty((rows, nh * 128), dtype=torch.uint8, device="cuda")
        fq = F.FusedQuant(q, scal[0:1], ws, F.E4M3, 0, bias_pred=scal[0:1], amax_bits=scal[1:2], flags=scal[2:3])
        o = torch.empty((rows, nh * 128), dtype=torch.bfloat16, device="cuda")
        F.llama_attention(qkv, case["seq"], nh, nkv, 128, o=o, fq=fq)
        return {"kind": "attention", "qkv": qkv, "seq": case["seq"], "nh": nh, "nkv": nkv, "o": o, "fq": fq, "scal": scal}
    k, n = case["k"], case["n"]
    w = _randn(_gen(seed), k, n, 0.01, torch.float32 if case["dtype"] == "f32" else torch.bfloat16)
    u8 = dict(dtype=torch.uint8, device="cuda")
    return {"kind": "ptq", "w": w, "w8": torch.empty((k, n), **u8), "w8t": torch.empty((n, k), **u8),
            "bw": torch.zeros(1, dtype=torch.int32, device="cuda"), "flags": torch.zeros(1, dtype=torch.int32, device="cuda"),
            "ws": F.workspace(k * n, "cuda")}


def _amax(scal):
    """[bias, amax bits, flags] with the amax as the fp32 value it is."""
    return {"bias": scal[0:1], "amax": scal[1:2].view(torch.float32), "flags": scal[2:3]}


def run(state):
    kind = state["kind"]
    if kind == "calls":
        b = state["b"]
        y, dx, dw = L.train_step(state["x"], state["w"], state["dy"], b)
        return {"y": y, "dx": dx, "dw": dw, "x8": b.x8, "x8t": b.x8t, "w8": b.w8, "w8t": b.w8t, "dy8": b.dy8, "dy8t": b.dy8t,
                "biases": b.scal[0:5], "flags": b.scal[10:15], "amax": b.scal[5:8].view(torch.float32)}
    if kind == "step":
        step = state["step"]
        step.replay()
        out = {}
        for name, qt in step.q.items():
            if not step.w.train and name.startswith("W"):
                continue                 # quantised at load
            out[name] = {"q": qt.q, "qT": qt.qT, **_amax(qt.scal)}
        for name, (hist, count) in step.hist.items():
            out["history " + name] = {"amax": hist.view(torch.float32), "count": count}
        for name, o in step.out.items():
            out[name] = {"y": o["y"]}
            if step.w.train:
                # the biases of the outputs (their amax moves with the rounding of one value)
                out[name].update(dx=o["dx"], dw=o["dw"], y_bias=o["y_scal"][0::2], dx_bias=o["dx_scal"][0::2])
        return out
    if kind == "layer":
        y = state["layer"]
        y.replay()
        acts = {"xn": y.xn, "att": y.att, "hn": y.hn, "act": y.act}
        out = {name: a.x for name, a in acts.items()}
        out.update(qkv=y.qkv, o=y.o, h1=y.h1, gu=y.gu, down=y.down, out=y.out)
        out["biases"] = {name: (a.seg_bias if y.bias_per == "sequence" else a.bias) for name, a in acts.items()}
        return out
    if kind == "attention":
        F.llama_attention(state["qkv"], state["seq"], state["nh"], state["nkv"], 128, o=state["o"], fq=state["fq"])
        return {"o": state["o"], **_amax(state["scal"])}
    F.ptq_quantise_weights(state["w"], w8=state["w8"], w8t=state["w8t"], bw=state["bw"], flags=state["flags"], ws=state["ws"])
    return {"w8": state["w8"], "w8t": state["w8t"], "bw": state["bw"], "flags": state["flags"]}


# ------------------------------------------------------------------ work
def _att_flops(rows, seq, nh):
    return 4 * nh * 128 * sum(min(seq, rows - s) * (min(seq, rows - s) + 1) // 2 for s in range(0, rows, seq))


def work(case):
    kind = case["kind"]
    if kind == "train":
        m, k, n = case["m"], case["k"], case["n"]
        # bf16 x, w, dy in; codes and transposed codes of each, bf16 y and dx, fp32 dw out
        return {"bytes": 4 * (m * k + k * n + m * n) + 2 * (m * n + m * k) + 4 * k * n, "flops": 6 * m * k * n}
    if kind == "serve":
        m = case["m"]
        return {"bytes": sum(k * n + 3 * m * k + 2 * m * n for _, k, n, _ in _linears(case)),
                "flops": sum(2 * m * k * n for _, k, n, _ in _linears(case))}
    if kind == "layer":
        d, nh, nkv, ffn, _ = MODELS[case["model"]]
        r = case["rows"]
        acts = [d, (nh + 2 * nkv) * 128, nh * 128, d, d, d, 2 * ffn, ffn, d, d]  # bf16 tensors of the layer
        return {"bytes": sum(k * n for _, k, n, _ in _linears(case)) + 2 * r * d + 2 * r * sum(acts),
                "flops": sum(2 * r * k * n for _, k, n, _ in _linears(case)) + _att_flops(r, case["seq"], nh)}
    if kind == "attention":
        _, nh, nkv, _, _ = MODELS[case["model"]]
        r = case["rows"]
        return {"bytes": 2 * r * (nh + 2 * nkv) * 128 + 3 * r * nh * 128, "flops": _att_flops(r, case["seq"], nh)}
    return {"bytes": (6 if case["dtype"] == "f32" else 4) * case["k"] * case["n"], "flops": 0}


def tolerance(case):
    kind = case["kind"]
    if kind in ("train", "serve"):
        # sums of another order in fp32, then one rounding to bf16: a value that
        # rounds the other way is off by one bf16 step (up to 2^-7 of it).  Four
        # times what the products differ by from the rounded fp64 ones (rel
        # 4.3e-4 with outlier channels, 2.3e-4 without; largest 7.8e-3)
        return {"rel": 1.7e-3, "max": 0.03}
    if kind == "layer":
        # a value that rounds the other way before a cast moves a code by one
        # E4M3 step: relative differences of about 1e-2 at the layer's end
        return {"rel": 0.03, "max": 1 - 1e-9}
    if kind == "attention":
        # probabilities rounded to bf16 before the product with V
        return {"rel": 0.008, "max": 0.1}
    return "exact"


# ------------------------------------------------------------------ exact
_MAX = {F.E4M3: 448.0, F.E5M2: 57344.0}
_T8 = {F.E4M3: torch.float8_e4m3fn, F.E5M2: torch.float8_e5m2}


def _bias(amax, fmt):
    """Largest integer b with amax 2^b <= the largest finite value (0 for amax 0)."""
    a = float(amax)
    if a == 0.0 or not math.isfinite(a):
        return 0
    b = math.frexp(_MAX[fmt])[1] - math.frexp(a)[1]
    return b if math.ldexp(a, b) <= _MAX[fmt] else b - 1


def _quant(x, fmt):
    """The FP8 values of x 2^b divided by 2^b, in fp64."""
    b = _bias(x.abs().max(), fmt)
    q = (x.double() * 2.0 ** b).float().to(_T8[fmt]).double()
    return q.mul_(2.0 ** -b)


def _bf(x):
    return x.float().to(torch.bfloat16).double()


def _attend(qkv, seq, nh, nkv):
    rows = qkv.shape[0]
    o = torch.empty((rows, nh * 128), dtype=torch.float64, device=qkv.device)
    for s in range(0, rows, seq):
        t = qkv[s:s + seq].double()
        n = t.shape[0]
        mask = torch.ones((n, n), dtype=torch.bool, device=qkv.device).triu_(1)
        for h in range(nh):
            hk = h // (nh // nkv)
            q, k, v = (t[:, c * 128:(c + 1) * 128] for c in (h, nh + hk, nh + nkv + hk))
            p = torch.softmax((q @ k.t() / math.sqrt(128.0)).masked_fill_(mask, -math.inf), 1)
            o[s:s + n, h * 128:(h + 1) * 128] = p @ v
    return o


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        x, w, dy = _train_inputs(case, seed)
        x, w, dy = _quant(x, F.E4M3), _quant(w, F.E4M3), _quant(dy, F.E5M2)
        out = {"y": x @ w, "dx": dy @ w.t(), "dw": x.t() @ dy}
        return out if case["quant"] == "calls" else {"linear": out}
    if kind == "serve":
        t = _serve_inputs(case, seed)
        return {name: {"y": _quant(t["X" + name], F.E4M3) @ _quant(t["W" + name], F.E4M3)} for name, _, _, _ in _linears(case)}
    if kind == "layer":
        return _exact_layer(case, seed)
    if kind == "attention":
        _, nh, nkv, _, _ = MODELS[case["model"]]
        return {"o": _attend(_attention_inputs(case, seed), case["seq"], nh, nkv)}
    return None


def _exact_layer(case, seed):
    w, h = _layer_inputs(case, seed)
    d, nh, nkv, ffn, _ = MODELS[case["model"]]
    seq, rows = case["seq"], case["rows"]

    def act(x):
        if case["per"] == "tensor":
            return _quant(x, F.E4M3)
        return torch.cat([_quant(x[s:s + seq], F.E4M3) for s in range(0, rows, seq)])

    def linear(x, key):
        return act(x) @ _quant(w[key], F.E4M3)

    def norm(x, g):
        return x / torch.sqrt((x * x).mean(1, keepdim=True) + D.LLAMA_EPS) * g.double()

    out = {}
    h = h.double()
    out["xn"] = norm(h, w["g_attn"])
    qkv = _bf(linear(_bf(out["xn"]), "Wqkv"))
    pos = (torch.arange(rows, device="cuda") % seq).double()
    ang = pos[:, None] * D.ROPE_THETA ** (-torch.arange(64, device="cuda").double() / 64.0)
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    rot = qkv[:, :(nh + nkv) * 128].view(rows, nh + nkv, 2, 64)
    a, b = rot[:, :, 0].clone(), rot[:, :, 1].clone()
    rot[:, :, 0], rot[:, :, 1] = a * cos - b * sin, b * cos + a * sin
    out["qkv"] = qkv
    out["att"] = _attend(_bf(qkv), seq, nh, nkv)
    out["o"] = linear(_bf(out["att"]), "Wo")
    out["h1"] = h + _bf(out["o"])
    h1 = _bf(out["h1"])
    out["hn"] = norm(h1, w["g_mlp"])
    out["gu"] = linear(_bf(out["hn"]), "Wgu")
    gate, up = _bf(out["gu"]).split(ffn, 1)
    out["act"] = gate * torch.sigmoid(gate) * up
    out["down"] = linear(_bf(out["act"]), "Wd")
    out["out"] = h1 + _bf(out["down"])
    return out
