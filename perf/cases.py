"""The work a program has this library do, as cases that can be timed and compared.

The unit is one GPU's share of one expert-parallel MoE layer (gate and top-k, routing
statistics, packaging, expert FFNs, combine), run through LayerShare at the model shapes
the repository configures, from one token to the largest prefill batch, and beside it the
FP8 routing predictor, which ranks a batch's experts ahead of the layer.

Serving programs replay short steps from a HIP graph (the layer allocates nothing and
never synchronises), so cases of up to GRAPH_MAX_T tokens and the predictor are captured
once in prepare() and replayed by run(); longer batches are enqueued call by call.
"""
from __future__ import annotations

import math
from typing import Dict

import numpy as np
import torch

from paper_2607_08782_amd import moe, synth
from paper_2607_08782_amd.layer import LayerShare

GRAPH_MAX_T = 1024
CHUNK = 2048          # rows of one 64-bit product in exact()

# the parity layer in 32 bits (64 tokens as configured) and the same kind of layer over an
# ordinary batch: what a program runs to check its numerics against
FP32_BATCH = dict(d=256, E=8, k=2, f=512)


def listed():
    return [
        # prompt processing, 2 of 8 wide experts here: the largest products
        {"name": "mixtral_prefill", "kind": "layer", "config": "mixtral_8x7b", "T": 4096},
        # one odd-sized chunk of a prompt: groups of a few dozen to a few hundred rows
        {"name": "mixtral_chunk", "kind": "layer", "config": "mixtral_8x7b", "T": 777},
        # a decode step over 64 running sequences: bound by the weights it reads
        {"name": "mixtral_decode", "kind": "layer", "config": "mixtral_8x7b", "T": 64},
        # prompt processing with many narrow experts, replicas and two shared experts
        {"name": "deepseek_prefill", "kind": "layer", "config": "deepseek_v2_lite", "T": 8192},
        # a decode step over 256 running sequences, shared experts in the routed call
        {"name": "deepseek_decode", "kind": "layer", "config": "deepseek_v2_lite", "T": 256},
        # one sequence decoding alone: the smallest step, launches and latency
        {"name": "deepseek_single", "kind": "layer", "config": "deepseek_v2_lite", "T": 1},
        # a batch of the drift sequence: one wide shared expert beside 8 narrow ones
        {"name": "qwen15_batch", "kind": "layer", "config": "qwen15_moe_a27b", "T": 2048},
        # the longest batch, 128 experts, top-8, co-activation counts
        {"name": "qwen3_prefill", "kind": "layer", "config": "qwen3_30b_a3b", "T": 16384},
        # its decode step: many launches over little data
        {"name": "qwen3_decode", "kind": "layer", "config": "qwen3_30b_a3b", "T": 64},
        # the 32-bit parity layer as configured
        {"name": "fp32_tiny", "kind": "layer", "config": "tiny_fp32", "T": 64},
        # a 32-bit layer over an ordinary, odd-sized batch
        {"name": "fp32_batch", "kind": "layer", "config": "fp32_batch", "T": 1000},
        # the quantized predictor ranking the experts of a batch: quantize, scores, top-k
        {"name": "predictor", "kind": "predictor", "config": "qwen3_30b_a3b", "T": 8192},
    ]


# longest batch drawn per configuration (the configured regimes' own)
_MAX_T = {"mixtral_8x7b": 4096, "deepseek_v2_lite": 8192, "qwen15_moe_a27b": 4096,
          "qwen3_30b_a3b": 16384, "tiny_fp32": 1024, "fp32_batch": 1024}


def draw(rng):
    kind = "predictor" if rng.random() < 0.15 else "layer"
    names = sorted(_MAX_T)
    if kind == "predictor":
        names = [n for n in names if not n.endswith("fp32") and not n.startswith("fp32")]
    name = rng.choice(names)
    T = int(round(math.exp(rng.uniform(0.0, math.log(_MAX_T[name])))))
    return {"kind": kind, "config": name, "T": T}


def _config(case) -> synth.LayerConfig:
    if case["config"] == "fp32_batch":
        return synth.custom_config(name="fp32_batch", dtype="f32", T=case["T"], **FP32_BATCH)
    return synth.CONFIGS[case["config"]]


def _inputs(case, seed: int) -> synth.LayerInputs:
    cfg = _config(case)
    experts = "none" if case["kind"] == "predictor" else "local"
    return synth.make_layer(cfg, case["T"], seed=seed, device="cuda", experts=experts)


class _State:
    """What the program keeps: the step to run, its outputs, and the graph it replays."""

    def __init__(self, step, outputs: Dict[str, torch.Tensor], keep, graph: bool):
        self.step, self.outputs, self.keep, self.graph = step, outputs, keep, None
        if graph:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                step()
            torch.cuda.current_stream().wait_stream(side)
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                step()
            self.graph = g


def _prepare_layer(case, seed: int) -> _State:
    inp = _inputs(case, seed)
    cfg = inp.cfg
    share = LayerShare(inp.X, inp.Wr, inp.bias, cfg.k, inp.placement, inp.dev, inp.w13, inp.w2,
                       shared=inp.shared, coact=cfg.coact)
    outputs = {"logits": share.logits, "topk_idx": share.topk_idx, "topk_gate": share.topk_gate,
               "counts": share.counts, "send_counts": share.perm["send_counts"], "y": share.y}
    if cfg.coact:
        outputs["coact"] = share.coact
    return _State(share.run, outputs, share, case["T"] <= GRAPH_MAX_T)


def _prepare_predictor(case, seed: int) -> _State:
    inp = _inputs(case, seed)
    cfg, T, dev = inp.cfg, case["T"], inp.X.device
    wq, ws = moe.moe_quantize_e4m3(inp.Wr)          # the replica's weights: quantized once
    out = {"q": torch.empty((T, cfg.d), dtype=torch.uint8, device=dev),
           "scales": torch.empty((T,), dtype=torch.float32, device=dev),
           "logits": torch.empty((T, cfg.E), dtype=torch.float32, device=dev),
           "topk_idx": torch.empty((T, cfg.k), dtype=torch.int32, device=dev),
           "topk_gate": torch.empty((T, cfg.k), dtype=torch.float32, device=dev)}

    def step():
        moe.moe_quantize_e4m3(inp.X, q=out["q"], scales=out["scales"])
        moe.moe_route_topk_e4m3(out["q"], out["scales"], wq, ws, inp.bias, cfg.k,
                                logits=out["logits"], topk_idx=out["topk_idx"],
                                topk_gate=out["topk_gate"])

    return _State(step, out, (inp, wq, ws), True)


def prepare(case, seed):
    return _prepare_predictor(case, seed) if case["kind"] == "predictor" else _prepare_layer(case, seed)


def run(state):
    if state.graph is not None:
        state.graph.replay()
    else:
        state.step()
    return state.outputs


def _expected_rows(cfg: synth.LayerConfig, T: int):
    """Rows and active experts this GPU can expect: the popularity bias over 4096 sampled
    score rows (the gate scores' own spread), the benchmark's placement."""
    rng = np.random.RandomState(1)
    pi = np.arange(cfg.E)
    bias = synth.zipf_bias(cfg, pi).astype(np.float64)
    place = synth.placement_map(cfg, pi)
    s = rng.standard_normal((4096, cfg.E)) * synth.WEIGHT_STD * math.sqrt(cfg.d) + bias
    top = np.argpartition(-s, cfg.k - 1, axis=1)[:, :cfg.k]
    p = np.bincount(top.reshape(-1), minlength=cfg.E) / 4096.0      # tokens per expert
    local = place[:, 0] != 0
    share = p / place.sum(1)                                       # replicas halve it
    rows = float((T * share)[local].sum())
    active = float((1.0 - (1.0 - np.minimum(share[local], 1.0)) ** T).sum())
    return rows, active


def work(case):
    cfg, T = _config(case), case["T"]
    size = 4 if cfg.dtype == "f32" else 2
    out = T * cfg.E * 4 + T * cfg.k * 8                            # scores, top-k, gates
    if case["kind"] == "predictor":
        return {"bytes": T * cfg.d * (size + 1) + T * 4 + cfg.E * (cfg.d + 8) + out,
                "flops": 2.0 * T * cfg.d * cfg.E}
    rows, active = _expected_rows(cfg, T)
    shared = sum(cfg.shared_f)
    weights = 3 * cfg.d * (active * cfg.f + shared) * size
    counts = 4 * cfg.E * (1 + (cfg.E if cfg.coact else 0)) + 4 * cfg.G
    return {"bytes": 2 * T * cfg.d * size + cfg.E * (cfg.d * size + 4) + weights + out + counts,
            "flops": 2.0 * T * cfg.d * cfg.E + 6.0 * cfg.d * (rows * cfg.f + T * shared)}


def tolerance(case):
    cfg = _config(case)
    # 32-bit sums in another order; whole values: an expert whose score ties with the next
    # to the last bits
    if case["kind"] == "predictor" or cfg.dtype == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
    # h and the expert outputs are rounded to bf16 on the way to y
    return {"rel": 1e-2, "max": 0.1, "differ": 5e-3}


def _mm(a, b):
    return torch.cat([a[i:i + CHUNK] @ b for i in range(0, a.shape[0], CHUNK)]) if len(a) else a @ b


def _swiglu(x, w13, w2):
    w13, w2 = w13.double(), w2.double()
    f = w2.shape[1]
    a, b = _mm(x, w13[:f].t().contiguous()), _mm(x, w13[f:].t().contiguous())
    return _mm(torch.nn.functional.silu(a) * b, w2.t().contiguous())


def _top(logits, k):
    val, idx = torch.topk(logits, k, dim=1)
    return idx, torch.softmax(val, dim=1)


def _exact_layer(case, seed: int):
    inp = _inputs(case, seed)
    cfg = inp.cfg
    x = inp.X.double()
    logits = _mm(x, inp.Wr.double().t().contiguous()) + inp.bias.double()
    idx, gate = _top(logits, cfg.k)
    y = torch.zeros_like(x)
    for e, w13, w2 in zip(inp.local, inp.w13, inp.w2):
        tok, rank = torch.nonzero(idx == e, as_tuple=True)         # ascending tokens
        hosts = [j for j in range(cfg.G) if inp.placement[e, j]]
        q, n, c = hosts.index(inp.dev), len(hosts), int(tok.numel())
        lo, hi = q * c // n, (q + 1) * c // n                      # this host's share
        tok, rank = tok[lo:hi], rank[lo:hi]
        if len(tok):
            y[tok] += gate[tok, rank].unsqueeze(1) * _swiglu(x[tok], w13, w2)
    for w13, w2 in inp.shared:
        y += _swiglu(x, w13, w2)
    return {"logits": logits, "topk_idx": None, "topk_gate": gate, "counts": None,
            "send_counts": None, "y": y, **({"coact": None} if cfg.coact else {})}


def _e4m3(w):
    """Codes' values and scales of a row-wise E4M3 quantization: 32-bit divisions, rounded
    from 64 bits (which is correctly rounded), then ties to even."""
    m = w.double().abs().amax(dim=1)
    s = torch.where(m > 0, m / 448.0, torch.ones_like(m)).float().double()
    q = (w.double() / s.unsqueeze(1)).float().clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return q.double(), s


def _exact_predictor(case, seed: int):
    inp = _inputs(case, seed)
    xq, xs = _e4m3(inp.X)
    wq, ws = _e4m3(inp.Wr)
    logits = _mm(xq, wq.t().contiguous()) * xs.unsqueeze(1) * ws + inp.bias.double()
    return {"q": None, "scales": xs, "logits": logits, "topk_idx": None,
            "topk_gate": _top(logits, inp.cfg.k)[1]}


def exact(case, seed):
    """What run() returns in 64 bits, by plain torch (no code of the library's)."""
    return _exact_predictor(case, seed) if case["kind"] == "predictor" else _exact_layer(case, seed)
