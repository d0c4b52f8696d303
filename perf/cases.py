"""The work that a user of this library has it do, as cases that can be timed.

Three kinds of pass, each through the public binding:

  linear   one W4A4 linear layer, basq_linear_fused, with what a serving program keeps per layer: the weights in the
           weight-streaming layout for decode-sized calls and in the fp6 operand form for longer ones.  The token count
           goes from one decoded token over batched and speculative decoding (tens of tokens) and short prompts
           (hundreds) to a long prefill.
  grouped  the same layer with activations quantised in groups of 128 channels: basq_rotate_quant with group_size = 128,
           then basq_w4a4_gemm_grouped.
  heads    the per-head rotation and quantiser of q, k and the KV cache: basq_rotate_quant with
           rot_size = group_size = 128.

Layer widths are those of `synth_inputs.CONFIGS` and of the tests: K = 1024, 4096, 8192 (one Sylvester rotation over the
whole token), 14336 (28 * 512) and 11008 (rotated in blocks of 256); N from 1024 to 28672.
"""
from __future__ import annotations

import math

import torch

from paper_2506_15689_amd import binding as B

# input width -> (rotation size, range clip ratio, outlier channels, their amplitude, standard deviation of the weights)
WIDTHS = {
    1024: (1024, 0.9, 8, 20.0, 0.02),
    4096: (4096, 0.9, 16, 20.0, 0.02),
    8192: (8192, 0.9, 32, 20.0, 0.015),
    11008: (256, 0.9, 32, 20.0, 0.02),
    14336: (14336, 0.85, 32, 30.0, 0.02),
}
HEAD = 128
MAX_PRODUCT = 4096 * 8192 * 28672          # M * K * N of the largest listed case
CALIBRATION_TOKENS = 512


def _linear(name, M, K, N, act_scale=False):
    return {"name": name, "kind": "linear", "M": M, "K": K, "N": N, "act_scale": act_scale}


def listed():
    return [
        # one token through a square projection: the smallest call of autoregressive decoding, all latency
        _linear("decode_1", 1, 4096, 4096),
        # the same projection with sixteen sequences decoded together
        _linear("decode_16", 16, 4096, 4096),
        # a few sequences through the widest layer: one pass over 117 MB of weights
        _linear("decode_wide_4", 4, 8192, 28672),
        # a small model's layer with a small batch
        _linear("small_layer_64", 64, 1024, 1024),
        # batched / speculative decoding, a ragged number of tokens, on a fused QKV projection
        _linear("batch_61", 61, 4096, 12288),
        # a short prompt, ragged, with the per-channel scale s^a of Eq. 15
        _linear("short_prompt_333", 333, 4096, 4096, act_scale=True),
        # fused QKV of a prefill
        _linear("qkv_prefill", 2048, 4096, 12288),
        # MLP down projection whose width needs the 28 * 512 rotation
        _linear("down_prefill", 2048, 14336, 4096),
        # MLP down projection rotated in blocks of 256, ragged prompt
        _linear("down_blockwise_1021", 1021, 11008, 4096),
        # gate/up projection of a long prefill: the largest call
        _linear("gate_up_prefill", 4096, 8192, 28672),
        # prefill with one activation range per 128 channels
        {"name": "grouped_prefill", "kind": "grouped", "M": 2048, "K": 4096, "N": 12288},
        # keys (or values, queries) of a prefill on their way into an INT4 KV cache, 32 heads of 128 channels
        {"name": "kv_heads", "kind": "heads", "M": 8192, "K": 4096},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges.  Token counts are spread over their logarithm and are mostly odd or ragged;
    output widths are multiples of 16, as model widths are."""
    pick = rng.random()
    if pick < 0.12:
        return {"kind": "heads", "M": _log_uniform(rng, 16, 16384), "K": rng.choice([1024, 2048, 4096, 8192])}
    N = 16 * _log_uniform(rng, 1024 // 16, 28672 // 16)
    if pick < 0.24:
        K = rng.choice([4096, 8192])
        most = min(4096, MAX_PRODUCT // (3 * K * N))            # a group costs about three times its share of the product
        return {"kind": "grouped", "M": _log_uniform(rng, 16, most), "K": K, "N": N}
    K = rng.choice([1024, 4096, 4096, 8192, 8192, 11008, 14336])
    most = min(4096, MAX_PRODUCT // (K * N))
    return {"kind": "linear", "M": _log_uniform(rng, 1, most), "K": K, "N": N, "act_scale": rng.random() < 0.25}


def _activations(gen, tokens, mu, scale):
    x = torch.randn((tokens, mu.numel()), generator=gen, device="cuda")
    return x.add_(mu).mul_(scale).to(torch.bfloat16)


def prepare(case, seed):
    kind, M, K = case["kind"], case["M"], case["K"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) + 20250615)
    rot, clip, n_out, amp, w_std = WIDTHS.get(K, (K, 0.9, 16, 20.0, 0.02))
    if kind == "heads":
        rot = HEAD
    # channels with different means, a few of them of much larger amplitude
    mu = torch.randn(K, generator=gen, device="cuda") * 0.5
    scale = torch.ones(K, device="cuda")
    scale[torch.randperm(K, generator=gen, device="cuda")[:n_out]] = amp
    X = _activations(gen, M, mu, scale)
    act_scale = None
    if case.get("act_scale"):
        act_scale = torch.exp(0.25 * torch.randn(K, generator=gen, device="cuda"))
    bias = torch.empty(K, device="cuda")
    cal = _activations(gen, CALIBRATION_TOKENS, mu, scale)
    B.basq_calibrate_bias(cal, rot, act_scale, bias, torch.empty(CALIBRATION_TOKENS * K, device="cuda"))
    s = {"kind": kind, "X": X, "rot": rot, "clip": clip, "bias": bias, "act_scale": act_scale}

    if kind == "heads":
        s["Aq"] = torch.empty((M, K // 2), dtype=torch.uint8, device="cuda")
        s["meta"] = torch.empty((M * (K // HEAD), 4), dtype=torch.int32, device="cuda")
        # step and lower bound, and row sum, of the 16-byte records (the fourth word is reserved)
        s["out"] = (s["Aq"], s["meta"].view(torch.float32)[:, :2], s["meta"][:, 2])
        return s

    N = case["N"]
    W = torch.randn((N, K), generator=gen, device="cuda").mul_(w_std).to(torch.bfloat16)
    layer_bias = torch.randn(N, generator=gen, device="cuda") * 0.1
    Wq, w_scale, w_zero, w_sum = B.alloc_weight_buffers(N, K)
    B.basq_quantize_weights(W, Wq, w_scale, w_zero, w_sum)
    Wq6 = B.alloc_fp6_buffer(N, K)
    out_bias = torch.empty(N, device="cuda")
    B.basq_prepare_weights(Wq, w_scale, w_zero, bias, layer_bias, w_sum, out_bias, Wq6)
    s.update(N=N, w_scale=w_scale, w_zero=w_zero, w_sum=w_sum, out_bias=out_bias, Wq6=Wq6,
             Y=torch.empty((M, N), dtype=torch.bfloat16, device="cuda"))
    if kind == "grouped":
        s["Wq"] = Wq
        s["w_gsum"] = torch.empty((K // HEAD, N), dtype=torch.int32, device="cuda")
        B.basq_group_colsums(Wq, HEAD, s["w_gsum"])
        s["Aq"] = torch.empty((M, K // 2), dtype=torch.uint8, device="cuda")
        s["meta"] = torch.empty((M * (K // HEAD), 4), dtype=torch.int32, device="cuda")
        s["Aq6"] = B.alloc_fp6_buffer(M, K)
    else:
        s["Wd"] = torch.empty(B.basq_decode_bytes(N, K), dtype=torch.uint8, device="cuda")
        B.basq_pack_decode(Wq, s["Wd"])
        s["workspace"] = torch.empty(B.basq_workspace_bytes(M, K, N), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    kind = s["kind"]
    if kind == "linear":
        B.basq_linear_fused(s["X"], s["rot"], s["bias"], s["act_scale"], s["clip"], s["clip"], s["Wd"], s["w_scale"],
                            s["w_zero"], s["w_sum"], s["out_bias"], s["Y"], s["workspace"], Wq6=s["Wq6"],
                            w_layout=B.BASQ_W_DECODE16, N=s["N"])
        return s["Y"]
    if kind == "grouped":
        B.basq_rotate_quant(s["X"], s["rot"], s["bias"], None, s["clip"], s["clip"], s["Aq"], s["meta"], Aq6=s["Aq6"],
                            group_size=HEAD)
        B.basq_w4a4_gemm_grouped(s["Aq"], s["meta"], HEAD, s["Wq"], s["w_scale"], s["w_zero"], s["w_gsum"], s["out_bias"],
                                 s["Y"], Aq6=s["Aq6"], Wq6=s["Wq6"])
        return s["Y"]
    B.basq_rotate_quant(s["X"], HEAD, s["bias"], None, s["clip"], s["clip"], s["Aq"], s["meta"], group_size=HEAD)
    return s["out"]


def work(case):
    M, K = case["M"], case["K"]
    rot = HEAD if case["kind"] == "heads" else WIDTHS[K][0]
    # the rotation as butterflies (H_28: 27 additions per output), then scale, range and quantiser: about eight per channel
    stages = math.log2(rot) if rot != 14336 else 9 + 27
    flops = M * K * (stages + 8)
    if case["kind"] == "heads":
        return {"bytes": M * (2 * K + K // 2 + 16 * (K // HEAD)) + 4 * K, "flops": flops}
    N = case["N"]
    # activations, 4-bit weights, per-channel vectors, outputs; group-wise ranges also need the weights' group sums
    nbytes = 2 * M * K + N * K // 2 + 12 * N + 4 * K + 2 * M * N
    if case["kind"] == "grouped":
        nbytes += 4 * N * (K // HEAD)
    if case.get("act_scale"):
        nbytes += 4 * K
    return {"bytes": nbytes, "flops": 2 * M * N * K + flops}


def tolerance(case):
    # Measured against the rotation in fp64 (and the product in fp64 on the codes that follow from it).  Another order of
    # the rotation's fp32 sums moves about one code per million by one step, which shows as rel 1e-5 .. 1.6e-3 of the
    # layer's output, the larger the fewer the tokens; one moved code of a lone token is about half a standard deviation
    # of one of its K values, 7e-3 at K = 4096.  Per-head records: rel 5e-8, max 3e-7; 1.3e-6 of the code bytes and
    # 8e-5 of the row sums differ.
    if case["kind"] == "heads":
        return {"rel": 2e-7, "max": 1.2e-6, "differ": 4e-4}
    return {"rel": 1e-2}
