"""The work this package is measured on: tile-wise (TW) sparse GEMMs as a user's program calls them.

A case is one call (or, for a Transformer layer, one chain of calls) on one MI355X: a weight pruned to the TW pattern
and packed once, activations that are new on every call, and an output buffer the program keeps.  The shapes are those of
`paper_2008_13006_amd.workloads` (BERT-base, BERT-large, a lowered 3x3 convolution) at batch sizes from a single
row to a full batch, plus generic ragged ones.

Fields of a case
  op         "gemm" (row-major A and C), "gemm_t" (both transposed), "dense" (an unpruned weight), "layer" (the four
             weight GEMMs of an encoder layer of width K, feed-forward width N, chained on one stream)
  M, K, N    rows of A (tokens, pixels), inputs and outputs of the weight
  dtype, G   16-bit storage type, tile granularity
  sparsity   zeros / (K*N), pruned columns included; col_prune: share of columns pruned altogether
  skew       "spread" (a tile keeps between 0.4 and 1.9 times the mean number of rows) or "zipf" (a few tiles
             keep most rows, as global ranking leaves a large feed-forward pair)
  delta      share of the weight put back as an element-wise residual (the TEW hybrid), 0 for none
  bias, act  fused epilogue: bias addition and "none", "relu" or "gelu"
  relu_in    activations are the output of a ReLU (half of them zero)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2008_13006_amd import binding as tw
from paper_2008_13006_amd import workloads as W

_BASE = dict(op="gemm", dtype="f16", G=128, sparsity=0.75, col_prune=0.05, skew="spread", delta=0.0, bias=False, act="none",
             relu_in=False)
_MAX_BYTES = 2.0 * 32 * 56 * 56 * (2304 + 256)       # A and C of the lowered convolution
_MAX_FLOPS = 2.0 * 16384 * 768 * 3072                # the dense feed-forward GEMM


def _case(**kw):
    return {**_BASE, **kw}


def listed():
    return [
        # one request of one token: the latency of a call
        _case(name="one_row_768x768", M=1, K=768, N=768),
        # a short sequence through one projection, no column pruned, every tile half full
        _case(name="single_256x768x768", M=256, K=768, N=768, sparsity=0.5, col_prune=0.0, skew="const"),
        # a serving batch through the weight GEMMs of a BERT-base layer: fused QKV, attention output, the feed-forward pair
        _case(name="bert_base_layer_512", op="layer", M=512, K=768, N=3072, bias=True, act="gelu"),
        # the second feed-forward GEMM (long K) at an ordinary batch
        _case(name="ffn_down_2048x3072x768", M=2048, K=3072, N=768, bias=True),
        # the headline workload: first feed-forward GEMM of BERT-base, full batch (128 sequences of 128 tokens)
        _case(name="ffn_up_16384x768x3072", M=16384, K=768, N=3072),
        # the same on the paper's transposed layout, for networks that keep their activations transposed
        _case(name="ffn_up_t_16384x768x3072", op="gemm_t", M=16384, K=768, N=3072),
        # the feed-forward pair of BERT-large in bf16, skewed tiles, with the epilogues it has inside a layer
        _case(name="ffn_up_large_gelu_8192x1024x4096", M=8192, K=1024, N=4096, dtype="bf16", sparsity=0.875, col_prune=0.10,
              skew="zipf", bias=True, act="gelu"),
        _case(name="ffn_down_large_t_8192x4096x1024", op="gemm_t", M=8192, K=4096, N=1024, dtype="bf16", sparsity=0.875,
              col_prune=0.10, skew="zipf", bias=True),
        # a 3x3 convolution lowered to a GEMM: few columns, very many rows, activations behind a ReLU
        _case(name="conv_relu_100352x2304x256", M=32 * 56 * 56, K=9 * 256, N=256, G=64, col_prune=0.0, bias=True, act="relu",
              relu_in=True),
        # the TEW hybrid: one weight in a hundred put back outside the pattern
        _case(name="tew_ffn_up_16384x768x3072", M=16384, K=768, N=3072, delta=0.01),
        # a layer that was left unpruned
        _case(name="dense_16384x768x3072", op="dense", M=16384, K=768, N=3072),
        # nothing a multiple of anything: a pitch of C that is no multiple of a line, narrow tiles, a last tile of odd width
        _case(name="ragged_4321x1000x1234", M=4321, K=1000, N=1234, dtype="bf16", G=32, sparsity=0.6, col_prune=0.03),
    ]


def _log_int(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]; half of them multiples of 64 (where that is in range)."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if v >= 64 and rng.random() < 0.5:
        v = (v + 32) // 64 * 64
    return max(lo, min(hi, v))


def draw(rng):
    op = rng.choice(["gemm", "gemm", "gemm", "gemm_t", "gemm_t", "dense", "layer"])
    dtype = rng.choice(["f16", "bf16"])
    bias = rng.random() < 0.5
    act = rng.choice(["none", "relu", "gelu"]) if bias else "none"
    if op == "layer":
        width = 64 * rng.randint(4, 16)
        return _case(op=op, M=_log_int(rng, 1, 4096), K=width, N=4 * width, dtype=dtype, sparsity=round(rng.uniform(0.5, 0.9), 3),
                     bias=True, act="gelu")
    K, N = _log_int(rng, 128, 4608), _log_int(rng, 128, 4096)
    if op == "dense":
        sparsity = 0.0
        N = (N + 7) // 8 * 8
    else:
        sparsity = round(rng.uniform(0.5, 0.9), 3)
    density = 1.0 - sparsity
    m_max = int(min(_MAX_BYTES / (2.0 * (K + N)), _MAX_FLOPS / (2.0 * K * N * min(1.0, 2.0 * density)), 100352))
    case = _case(op=op, M=_log_int(rng, 1, m_max), K=K, N=N, dtype=dtype, G=rng.choice([32, 64, 128, 128]), sparsity=sparsity,
                 col_prune=round(rng.uniform(0.0, 0.10), 3), skew=rng.choice(["spread", "spread", "zipf", "const"]),
                 bias=bias, act=act, relu_in=rng.random() < 0.3)
    if op != "dense" and K * N <= 3 * 2 ** 20 and case["M"] <= 16384 and rng.random() < 0.25:
        case["delta"] = round(rng.uniform(0.002, 0.02), 4)
    return case


# ------------------------------------------------------------------------------------------------ inputs
def _torch_dtype(dtype):
    return torch.float16 if dtype == "f16" else torch.bfloat16


def _mask(abs_b, case, rng):
    """Columns of least L1 norm pruned first, the rest regrouped G at a time, every tile keeps its strongest rows."""
    K, N = abs_b.shape
    n_pruned = int(math.floor(case["col_prune"] * N + 0.5))
    T = -(-(N - n_pruned) // case["G"])
    f = (1.0 - case["sparsity"]) * N / (N - n_pruned)
    if case["skew"] == "const" or T < 4:
        keep, target = ("const", min(1.0, f)), None
    elif case["skew"] == "zipf":
        keep, target = ("zipf", 0.16 * f, min(1.0, 4.3 * f), 1.2), case["sparsity"]
    else:
        keep, target = ("upow", 0.4 * f, min(1.0, 1.9 * f)), case["sparsity"]
    return W.tw_mask_from_scores(abs_b, case["G"], case["col_prune"], keep, target, rng)[0]


def _weight(case, K, N, rng):
    """A packed weight on the GPU: N(0, 0.02) values pruned by magnitude, as `workloads` draws them."""
    bits = W.f32_to_bits(rng.standard_normal((K, N), dtype=np.float32) * np.float32(0.02), case["dtype"])
    abs_b = np.abs(W.bits_to_f32(bits, case["dtype"]).astype(np.float64))
    mask = _mask(abs_b, case, rng)
    if case["delta"] > 0:
        ew = tw.tw_restore_ew(bits, mask, case["delta"], case["dtype"])
        return tw.TwWeight(tw.tw_pack_tew(bits, mask, ew, case["G"], case["dtype"]))
    return tw.TwWeight(tw.tw_pack(bits, mask, case["G"], case["dtype"]))


def _matrix(rows, cols, dtype, gen=None, scale=1.0, relu=False, pitch=8):
    """rows x cols on the GPU, the row pitch a multiple of `pitch` elements; N(0, scale) values with a generator."""
    ld = -(-cols // pitch) * pitch
    if gen is None:
        return torch.empty((rows, ld), dtype=_torch_dtype(dtype), device="cuda")[:, :cols]
    out = torch.empty((rows, ld), dtype=_torch_dtype(dtype), device="cuda")
    step = max(1, 2 ** 26 // ld)
    for r in range(0, rows, step):
        v = torch.randn((min(step, rows - r), ld), generator=gen, device="cuda") * scale
        out[r:r + step] = v.clamp_(min=0.0) if relu else v
    return out[:, :cols]


def prepare(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    op, M, K, N, dtype = case["op"], case["M"], case["K"], case["N"], case["dtype"]
    st = {"op": op, "act": case["act"], "bias": None}
    if op == "layer":
        st["w"] = [_weight(case, k, n, rng) for k, n in ((K, 3 * K), (K, K), (K, N), (N, K))]
        st["biases"] = [_matrix(1, n, dtype, gen, 0.1)[0] for n in (3 * K, K, N, K)]
        st["A"] = _matrix(M, K, dtype, gen)
        st["out"] = [_matrix(M, n, dtype) for n in (3 * K, K, N, K)]
        st["head"] = st["out"][0][:, :K]
        return st
    if case["bias"]:
        st["bias"] = _matrix(1, N, dtype, gen, 0.1)[0]
    if op == "gemm_t":
        st["A"] = _matrix(K, M, dtype, gen, relu=case["relu_in"], pitch=64)
        st["C"] = _matrix(N, M, dtype, pitch=64)
    else:
        st["A"] = _matrix(M, K, dtype, gen, relu=case["relu_in"])
        st["C"] = _matrix(M, N, dtype, pitch=8 if op == "dense" else 1)
    st["w"] = _matrix(K, N, dtype, gen, 0.02) if op == "dense" else _weight(case, K, N, rng)
    return st


# ------------------------------------------------------------------------------------------------ one pass
def run(st):
    op, w, bias, act = st["op"], st["w"], st["bias"], st["act"]
    if op == "layer":
        qkv, att, hid, out = st["out"]
        b = st["biases"]
        tw.tw_gemm_bias_act(w[0], st["A"], b[0], "none", qkv)
        tw.tw_gemm_bias_act(w[1], st["head"], b[1], "none", att)
        tw.tw_gemm_bias_act(w[2], att, b[2], act, hid)
        tw.tw_gemm_bias_act(w[3], hid, b[3], "none", out)
        return st["out"]
    if op == "gemm_t":
        if bias is None:
            return tw.tw_gemm_t(w, st["A"], st["C"])
        return tw.tw_gemm_t_bias_act(w, st["A"], bias, act, st["C"])
    if op == "dense":
        if bias is None:
            return tw.tw_dense_gemm(st["A"], w, st["C"])
        return tw.tw_dense_gemm_bias_act(st["A"], w, bias, act, st["C"])
    if bias is None:
        return tw.tw_gemm(w, st["A"], st["C"])
    return tw.tw_gemm_bias_act(w, st["A"], bias, act, st["C"])


def work(case):
    """A (of a layer: every intermediate too) read once, the kept weights read once, every output written once."""
    M, K, N = case["M"], case["K"], case["N"]
    density = 1.0 - case["sparsity"] + case["delta"] if case["op"] != "dense" else 1.0
    shapes = ((K, 3 * K), (K, K), (K, N), (N, K)) if case["op"] == "layer" else ((K, N),)
    nbytes = sum(2.0 * M * (k + n) + 2.0 * density * k * n for k, n in shapes)
    if case["bias"]:
        nbytes += sum(2.0 * n for _, n in shapes)
    return {"bytes": nbytes, "flops": sum(2.0 * M * k * n * density for k, n in shapes)}


def tolerance(case):
    """Results are sums in fp32 rounded once to 16 bits."""
    return {"rel": 8e-4} if case["dtype"] == "f16" else {"rel": 7e-3}
