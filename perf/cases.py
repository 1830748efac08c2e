"""What a program that serves or loads a W6A6 / W6A8 model asks of this library, as cases that can be timed and compared.

Four kinds of work, each through the public calls of `paper_2508_04405_amd`:

  linear   one quantized linear layer with the activation quantizer that feeds it
  block    the seven linear layers of a decoder block with their fused producers (one `layer_linears` call)
  xgroup   one linear layer with group-128 scales on both operands
  pack     quantizing and packing a layer's weights when a checkpoint is loaded

Weights, workspace and output buffers are what such a program keeps; activations are new with every seed. Sizes are the
LLaMA-2 layer dimensions of the benchmark, one ragged size, and in `draw` sizes spread over the range that the calls accept.
"""
import math

import torch

import paper_2508_04405_amd as fq

# hidden size, feed-forward width, fused QKV width
MODELS = {"7b": (4096, 11008, 12288), "13b": (5120, 13824, 15360), "70b": (8192, 28672, 10240)}
EPS = 1e-5
SIGMA = 0.02                          # of the weights
MOST_MACS = 3.5e12                    # per pass: the 70B block at 4096 tokens
MOST_WEIGHTS = 8192 * 57344


def listed():
    return [
        # the smallest call: one token through LLaMA-2-7B's attention output projection, fp16 in, fp16 out
        dict(name="linear 7b o 1 token", kind="linear", feed="fp16", M=1, K=4096, N=4096, bits=8, group=0),
        # batched decode of a program with a norm of its own in front: LLaMA-2-70B's fused QKV at 16 tokens
        dict(name="linear 70b qkv 16 tokens", kind="linear", feed="norm", M=16, K=8192, N=10240, bits=6, group=0),
        # token generation, one request: a 70B decoder block, 6 bits and 8 on the down projection
        dict(name="block 70b 1 token", kind="block", model="70b", M=1, bits="6668", group=0),
        # token generation, eight requests: a 7B decoder block with 8-bit activations throughout
        dict(name="block 7b 8 tokens", kind="block", model="7b", M=8, bits="8888", group=0),
        # batched decode of the 13B stack, group-128 weight scales
        dict(name="block 13b g128 32 tokens", kind="block", model="13b", M=32, bits="6666", group=128),
        # a large decode batch or a short prompt: 70B's down projection behind the gated SiLU, an odd token count
        dict(name="linear 70b down 97 tokens", kind="linear", feed="swiglu", M=97, K=28672, N=8192, bits=8, group=0),
        # nothing a multiple of a tile: a prompt of 333 tokens on a layer of 427 row blocks and 41 groups
        dict(name="linear ragged 333 tokens", kind="linear", feed="fp16", M=333, K=5248, N=13664, bits=6, group=0),
        # a medium prompt: 70B's fused QKV at 1024 tokens
        dict(name="linear 70b qkv 1024 tokens", kind="linear", feed="fp16", M=1024, K=8192, N=10240, bits=6, group=0),
        # prefill with one scale per group on both operands: 13B's down projection at an odd token count
        dict(name="xgroup 13b down 700 tokens", kind="xgroup", M=700, K=13824, N=5120, bits=8),
        # prefill of the 13B stack, group-128 weight scales, a layer that runs 8 bits throughout
        dict(name="block 13b g128 2048 tokens", kind="block", model="13b", M=2048, bits="8888", group=128),
        # the largest: prefill of a 70B decoder block
        dict(name="block 70b 4096 tokens", kind="block", model="70b", M=4096, bits="6668", group=0),
        # loading a checkpoint: one 70B attention output projection quantized and packed
        dict(name="pack 70b o", kind="pack", N=8192, K=8192, group=0),
    ]


def _log_int(rng, low, high):
    return max(low, min(high, int(math.exp(rng.uniform(math.log(low), math.log(high + 1))))))


def draw(rng):
    kind = rng.choice(["linear"] * 5 + ["block"] * 3 + ["xgroup", "pack"])
    while True:
        if kind == "block":
            c = dict(kind=kind, model=rng.choice(sorted(MODELS)), M=_log_int(rng, 1, 4096),
                     bits=rng.choice(["6668", "8888", "6666"]), group=rng.choice([0, 0, 128]))
        elif kind == "pack":
            c = dict(kind=kind, N=128 * _log_int(rng, 4, 448), K=128 * _log_int(rng, 4, 224), group=rng.choice([0, 128]))
        else:
            if rng.random() < 0.5:
                H, F, QKV = MODELS[rng.choice(sorted(MODELS))]
                K, N = rng.choice([(H, QKV), (H, H), (H, 2 * F), (F, H)])
            else:
                K, N = 128 * _log_int(rng, 4, 224), 32 * _log_int(rng, 16, 1792)
            c = dict(kind=kind, M=_log_int(rng, 1, 4096), K=K, N=N, bits=rng.choice([6, 8]))
            if kind == "linear":
                c["group"] = rng.choice([0, 0, 128])
                c["feed"] = rng.choice(["fp16", "fp16", "norm", "swiglu"] + (["tiles"] if c["M"] <= 32 else []))
        grouped = kind == "xgroup" or c.get("group") == 128
        M, weights = c.get("M", 1), sum(k * n for k, n in _shapes(c))
        if (kind == "block" or weights <= MOST_WEIGHTS) and M * weights <= MOST_MACS * (0.3 if grouped else 1.0):
            return c


def _shapes(c):
    """(K, N) of every matrix product of a pass."""
    if c["kind"] != "block":
        return [(c["K"], c["N"])]
    H, F, QKV = MODELS[c["model"]]
    return [(H, QKV), (H, H), (H, 2 * F), (F, H)]


# ---- inputs, from the seed alone -------------------------------------------------------------------------------

class _Source:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def weights(self, N, K):
        return torch.randn((N, K), generator=self.g, device="cuda").mul_(SIGMA)

    def activations(self, M, K):
        """N(0, 1), one channel in a hundred twenty times as large for every token."""
        x = torch.randn((M, K), generator=self.g, device="cuda")
        x[:, torch.randperm(K, generator=self.g, device="cuda")[:max(1, K // 100)]] *= 20.0
        return x.half()

    def gate_up(self, M, F):
        """N(0, 1.5) with sparse large entries, as ahead of a down projection."""
        x = torch.randn((M, 2 * F), generator=self.g, device="cuda").mul_(1.5)
        return torch.where(torch.rand((M, 2 * F), generator=self.g, device="cuda") < 5e-4, 12.0 * x, x).half()

    def gain(self, K):
        return (1.0 + 0.1 * torch.randn(K, generator=self.g, device="cuda")).half()


def _inputs(c, seed):
    s = _Source(seed)
    if c["kind"] == "pack":
        return dict(w=s.weights(c["N"], c["K"]))
    M = c["M"]
    d = dict(w=[])
    if c["kind"] == "block":
        H = MODELS[c["model"]][0]
        d.update(x=s.activations(M, H), attn=s.activations(M, H), gamma_attn=s.gain(H), gamma_ffn=s.gain(H))
    elif c["kind"] == "linear" and c["feed"] == "swiglu":
        d["x"] = s.gate_up(M, c["K"])
    else:
        d.update(x=s.activations(M, c["K"]), gamma=s.gain(c["K"]))
    d["w"] = (s.weights(n, k) for k, n in _shapes(c))      # one at a time: they are large
    return d


def prepare(case, seed):
    c, d = case, _inputs(case, seed)
    if c["kind"] == "pack":
        return dict(case=c, w=d["w"])
    group = 128 if c["kind"] == "xgroup" else c["group"]
    packed = [fq.pack_w6(*fq.quant_w6(w, group), group) for w in d.pop("w")]
    M = c["M"]
    if c["kind"] == "block":
        H, F, QKV = MODELS[c["model"]]
        layer = fq.Layer(H, F, QKV, group, *packed, d["gamma_attn"], d["gamma_ffn"], EPS, tuple(int(b) for b in c["bits"]))
        outs = {k: torch.empty((M, n), dtype=torch.float16, device="cuda")
                for k, n in (("qkv", QKV), ("o", H), ("gate_up", 2 * F), ("down", H))}
        return dict(case=c, layer=layer, workspace=layer.make_workspace(M), x=d["x"], attn=d["attn"], outs=outs)
    K, N = c["K"], c["N"]
    s = dict(case=c, packed=packed[0], workspace=fq.make_workspace(M, N, K), x=d["x"], gamma=d.get("gamma"),
             out=torch.empty((M, N), dtype=torch.float16, device="cuda"))
    if c["kind"] == "linear" and c["feed"] in ("norm", "swiglu"):     # the codes' buffers, kept like the workspace
        s["codes"] = (torch.empty((M, K), dtype=torch.int8, device="cuda"),
                      torch.empty((M,), dtype=torch.float16, device="cuda"))
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "pack":
        wq, sw = fq.quant_w6(s["w"], c["group"])
        return dict(packed=fq.pack_w6(wq, sw, c["group"]), scales=sw)
    if c["kind"] == "block":
        outs = s["outs"]
        fq.layer_linears(s["layer"], c["M"], s["workspace"], x=s["x"], attn=s["attn"], x_ffn=outs["o"], **outs)
        return outs
    N, K, bits = c["N"], c["K"], c["bits"]
    if c["kind"] == "xgroup":
        xq, sxg = fq.quant_act_g128(s["x"], bits)
        return fq.linear_g128(s["packed"], N, K, xq, sxg, workspace=s["workspace"], out=s["out"])
    if c["feed"] == "tiles":
        xt, sx = fq.quant_act_tiles(s["x"], bits)
        return fq.gemv_tiles(bits, s["packed"], N, K, c["group"], xt, sx, workspace=s["workspace"], out=s["out"])
    if c["M"] <= 32:
        linear = fq.gemv_w6a6 if bits == 6 else fq.gemv_w6a8
    else:
        linear = fq.gemm_w6a6 if bits == 6 else fq.gemm_w6a8
    if c["feed"] == "fp16":
        return linear(s["packed"], N, K, c["group"], x_fp16=s["x"], workspace=s["workspace"], out=s["out"])
    if c["feed"] == "norm":
        xq, sx = fq.rmsnorm_quant(s["x"], s["gamma"], EPS, bits, out=s["codes"])
    else:
        xq, sx = fq.swiglu_quant(s["x"], bits, out=s["codes"])
    return linear(s["packed"], N, K, c["group"], xq=xq, sx=sx, workspace=s["workspace"], out=s["out"])


def work(case):
    """Every input read once, every output written once: fp16 activations in, packed weights and scales, fp16 out."""
    c = case
    if c["kind"] == "pack":
        weights = c["N"] * c["K"]
        scales = c["N"] * (c["K"] // 128 if c["group"] else 1)
        return dict(bytes=4.75 * weights + 4.0 * scales, flops=0)     # the scales come back twice: alone and packed
    M = c["M"]
    grouped = c["kind"] == "xgroup" or c["group"] == 128
    bytes_ = flops = 0.0
    for i, (K, N) in enumerate(_shapes(c)):
        bytes_ += 0.75 * N * K + 2.0 * N * (K // 128 if grouped else 1) + 2.0 * M * N
        flops += 2.0 * M * N * K
        if c["kind"] != "block":
            bytes_ += 2.0 * M * K * (2 if c.get("feed") == "swiglu" else 1)
        elif i < 2:
            bytes_ += 2.0 * M * K                                      # x and attn; the other stages read outputs
    return dict(bytes=bytes_, flops=flops)


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    if case["kind"] == "block" or case.get("feed") in ("norm", "swiglu"):
        # a producer's fp16 value that rounds the other way moves a code by one step, and a row's
        # largest value that does moves its scale
        return dict(rel=4e-3, max=0.1)
    return dict(rel=1e-3, max=4e-3)            # the codes are exact: fp16 results within one place


# ---- the same in 64 bits, in plain torch -------------------------------------------------------------------------

def _quantize(v, bits, group=0):
    """Symmetric codes and fp16 scales of rows (or of groups of 128 along them), both as 64-bit floats."""
    qmax = 2.0 ** (bits - 1) - 1
    v = v.double()
    rows, K = v.shape
    v = v.view(rows, K // (group or K), group or K)
    top = v.abs().amax(-1, keepdim=True)
    s = (top / qmax).float().half().double()
    s = torch.where((top == 0) | (s == 0), torch.ones_like(s), s)
    q = (v / s).float().double().round_().clamp_(-qmax - 1, qmax)     # the 32-bit quotient, half to even
    return q, s


def _dequantized(v, bits, group=0):
    q, s = _quantize(v, bits, group)
    return (q * s).view(v.shape)


def _norm(x, gamma):
    x = x.double()
    return (x / (x.square().mean(1, keepdim=True) + EPS).sqrt() * gamma.double()).half()


def _swiglu(x):
    g, u = x.double().chunk(2, 1)
    return (g / (1.0 + torch.exp(-g)) * u).half()


def exact(case, seed):
    c, d = case, _inputs(case, seed)
    if c["kind"] == "pack":
        return dict(packed=None, scales=_quantize(d["w"], 6, c["group"])[1].squeeze(-1) if c["group"]
                    else _quantize(d["w"], 6)[1].view(-1))
    if c["kind"] == "xgroup":
        return _dequantized(d["x"], c["bits"], 128) @ _dequantized(next(d["w"]), 6, 128).t()
    g = c["group"]
    if c["kind"] == "linear":
        h = d["x"] if c["feed"] in ("fp16", "tiles") else _norm(d["x"], d["gamma"]) if c["feed"] == "norm" else _swiglu(d["x"])
        return _dequantized(h, c["bits"]) @ _dequantized(next(d["w"]), 6, g).t()
    b, outs = [int(x) for x in c["bits"]], {}

    def linear(h, bits):
        return _dequantized(h, bits) @ _dequantized(next(d["w"]), 6, g).t()

    outs["qkv"] = linear(_norm(d["x"], d["gamma_attn"]), b[0])
    outs["o"] = linear(d["attn"], b[1])
    outs["gate_up"] = linear(_norm(outs["o"].half(), d["gamma_ffn"]), b[2])
    outs["down"] = linear(_swiglu(outs["gate_up"].half()), b[3])
    return outs
