"""The work whose time is kept track of: whole executions of compiled memgraphs through the public
entry points (harness.GpuSession: tiler, compiler and executor behind the C ABI), over the range of
shapes, storage types and tiler options that the repository's configurations, tests and benchmark use.

A case is one program: a decoder shape, what it does (prefill, prefill + decode steps, fine-tuning
step), the GPU-memory cap, where inputs and outputs live, and the options the benchmark would run that
kind of workload with.  `prepare` makes the inputs and the compiled, loaded program; `run` is one step.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2405_16283_amd import binding as B
from paper_2405_16283_amd import harness as H
from workloads import LlamaConfig

# What a case says where it says nothing else.
DEFAULTS = {
    "mode": "prefill",        # "prefill", "decode" (prefill, then `decode_steps` rows) or "train" (forward + reverse)
    "dtype": "bf16",
    "layers": 1,              # layers share one set of weights: same shapes, vertices and transfers
    "batch": 1,
    "decode_steps": 0,
    "cap_mb": 0,              # GPU-memory cap in MB ...
    "cap_pct": 0,             # ... or as a percentage of the uncapped peak working set
    "on_gpu": False,          # inputs placed in the capped buffer from GPU memory, results left in GPU memory
    "kv_outputs": False,
    "order": "tiler",         # serial order given to the compiler
    "pressed": False,         # compile options for a cap far below the working set
    "whole_rows": False,
    "fuse": 0,
    "materialize": False,
    "max_transfers": 0,
    "copy_workgroups": 0,
    "small_tiles": 0,
    "gemm_inflight": 1,
}
LORA_RANK = 16


def listed():
    return [
        # The smallest programs: latency and launches count.
        # The two-layer toy decoder under 40 % of its peak, everything on the host.
        dict(name="toy_f32", dtype="f32", layers=2, heads=4, head_dim=64, ffn=688, seq=128, tile=64, block=64, cap_pct=40),
        # Its fine-tuning step on ragged shapes (two sequences of 160 tokens, ffn 272), saved activations offloaded.
        dict(name="ragged_f32_train", mode="train", dtype="f32", layers=2, heads=3, head_dim=64, ffn=272, seq=160, batch=2,
             tile=64, block=128, cap_pct=40),
        # fp32 storage at a size where arithmetic counts.
        dict(name="prefill_f32", dtype="f32", heads=16, head_dim=64, ffn=2752, seq=1024, tile=256, block=512, cap_pct=60),
        # bf16 with ragged tiles (1152 = 3 x 384, 1440 = 3 x 384 + 288) under 40 % of the peak.
        dict(name="ragged_bf16_capped", heads=9, head_dim=128, ffn=1440, seq=1440, tile=384, block=768, cap_pct=40),
        # A 7B-shaped layer on a prompt whose length is no multiple of anything.
        dict(name="prompt_1371", heads=32, head_dim=128, ffn=11008, seq=1371, tile=512, block=1024, cap_mb=1500, on_gpu=True, fuse=3),
        # The same layer on 4096 tokens, everything in GPU memory: the tile kernels by themselves.
        dict(name="layer_4096", heads=32, head_dim=128, ffn=11008, seq=4096, tile=512, block=1024, cap_mb=2000, on_gpu=True, fuse=3),
        # The same streamed from the host under 40 % of its peak.
        dict(name="layer_4096_capped", heads=32, head_dim=128, ffn=11008, seq=4096, tile=512, block=1024, cap_pct=40,
             order="clustered", pressed=True, fuse=3, max_transfers=32, copy_workgroups=16, small_tiles=-1),
        # One layer of the long-sequence prefill (16384 tokens), weights streamed, keys and values stored to the host.
        dict(name="long_16384", heads=32, head_dim=128, ffn=11008, seq=16384, tile=512, block=1024, cap_mb=8000,
             order="clustered", whole_rows=True, fuse=3, kv_outputs=True),
        # One layer of the 65B shape, 8192 tokens: bound by its weights' way over the host link.
        dict(name="stream_65b", heads=64, head_dim=128, ffn=22016, seq=8192, tile=1024, block=1024, cap_mb=4000,
             kv_outputs=True, max_transfers=128, copy_workgroups=14, small_tiles=-1),
        # One layer of the fine-tuning step: rank-16 adapters, four sequences of 4096 tokens, forward and reverse pass.
        dict(name="finetune_4x4096", mode="train", heads=32, head_dim=128, ffn=11008, seq=4096, batch=4, tile=512, block=1024,
             cap_mb=12000, small_tiles=-1, gemm_inflight=2),
        # Generation: a prompt of 320 tokens and 32 single-row steps through two 7B-shaped layers, weights in GPU memory.
        dict(name="decode_32", mode="decode", layers=2, heads=32, head_dim=128, ffn=11008, seq=320, decode_steps=32, tile=512,
             block=1024, cap_mb=2500, on_gpu=True),
        # Attention with scores and probabilities as tensors of the graph (one head per column tile).
        dict(name="scores_2048", heads=16, head_dim=128, ffn=5504, seq=2048, tile=128, block=1024, cap_mb=1000, order="level",
             materialize=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another program of the same ranges: tiny to 7B-shaped layers, prompts of any length, both storage
    types, resident or streamed under a cap, prefill, decode, fine-tuning, fused or materialised attention."""
    mode = rng.choice(["prefill", "prefill", "prefill", "prefill", "train", "train", "decode", "decode", "scores"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    head_dim = rng.choice([64, 128, 128])
    width = _log_int(rng, 256, (1024 if mode == "scores" else 4096) if dtype == "bf16" else 1024)
    if mode == "scores":
        tile = head_dim
    else:  # 3 to 16 tiles across the model, as in the configurations
        tile = rng.choice([t for t in (64, 128, 256, 384, 512) if t % head_dim == 0 and 3 * t <= width <= 16 * t] or [head_dim])
    d_model = max(1, width // tile) * tile
    ffn = max(64, int(d_model * rng.uniform(1.25, 2.75)) // 16 * 16)
    seq = _log_int(rng, 96, {"prefill": 4096, "train": 2048, "decode": 1024, "scores": 1024}[mode] // (1 if dtype == "bf16" else 4))
    while mode == "train" and seq * d_model > 1 << 22:
        seq //= 2
    block = tile * rng.choice([1, 2, 2, 4])
    case = dict(mode="prefill" if mode == "scores" else mode, dtype=dtype, layers=rng.choice([1, 1, 2]), heads=d_model // head_dim,
                head_dim=head_dim, ffn=ffn, seq=seq, tile=tile, block=block)
    if mode == "scores":
        case.update(materialize=True, order="level")
    elif mode == "decode":
        case["decode_steps"] = rng.randint(4, 32)
    elif rng.random() < 0.4:
        case["batch"] = rng.choice([2, 3])
    if mode in ("prefill", "decode"):
        case.update(fuse=rng.choice([0, 3]), kv_outputs=rng.random() < 0.3, order=rng.choice(["tiler", "clustered"]))
    if rng.random() < 0.5 and mode != "train":
        case.update(on_gpu=True, cap_pct=rng.randint(150, 300))
        case["whole_rows"] = mode != "scores" and rng.random() < 0.4
    elif mode == "decode":
        case["cap_pct"] = rng.randint(110, 150)
    else:
        case["cap_pct"] = rng.randint(60 if seq >= 400 else 110, 140)  # a short program's largest vertex needs most of its peak
    return case


def _config(case):
    c = {**DEFAULTS, **case}
    cfg = LlamaConfig(c.get("name", "drawn"), c["layers"], c["heads"] * c["head_dim"], c["heads"], c["head_dim"], c["ffn"], c["seq"],
                      c["batch"], c["dtype"], c["tile"], c["block"], c["cap_mb"] * 10**6, c["cap_pct"] / 100.0, c["on_gpu"],
                      c["on_gpu"], decode_steps=c["decode_steps"])
    return c, cfg


def _tiler_options(c):
    train = c["mode"] == "train"
    return dict(kv_outputs=c["kv_outputs"], lora_rank=LORA_RANK if train else 0, train=train, materialize_scores=c["materialize"],
                attn_whole_rows=c["whole_rows"], fuse_epilogues=c["fuse"], recompute_normed=train, recompute_gate_up=train)


def _inputs(cfg, c, seed):
    """Full tensors in storage type, as workloads.make_llama_inputs / make_lora_inputs would lay them out
    (weights N(0, 0.02), x and probe N(0, 1), gains 1 + 0.02 N(0, 1), adapters N(0, 0.02)), drawn on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    kind = torch.float32 if cfg.dtype == "f32" else torch.bfloat16

    def tensor(shape, std, mean=0.0):
        t = torch.randn(shape, generator=g, device="cuda", dtype=kind).mul_(std)
        a = (t.add_(mean) if mean else t)
        return a.cpu().numpy() if cfg.dtype == "f32" else a.view(torch.int16).cpu().numpy().view(np.uint16)

    d, f = cfg.d_model, cfg.ffn
    full = {"x": tensor((cfg.tokens, d), 1.0)}
    one = {k: tensor((o, i), 0.02).T for k, i, o in (("wq", d, d), ("wk", d, d), ("wv", d, d), ("wo", d, d), ("w1", d, f),
                                                     ("w3", d, f), ("w2", f, d))}  # stored [out, in], as checkpoints are
    one.update({k: tensor((d,), 0.02, 1.0) for k in ("g1", "g2")})
    if c["mode"] == "train":
        full["probe"] = tensor((cfg.tokens, d), 1.0)
        one.update({k: tensor((d, LORA_RANK), 0.02) for k in ("aq", "av")})
        one.update({k: tensor((LORA_RANK, d), 0.02) for k in ("bq", "bv")})
    for layer in range(cfg.layers):
        full.update({f"{k}.{layer}": a for k, a in one.items()})
    return full


class Program:
    """A compiled and loaded program with its inputs: what a caller keeps between steps."""

    def __init__(self, case, seed):
        c, cfg = _config(case)
        train = c["mode"] == "train"
        if not cfg.cap_bytes:
            tg = B.tn_build_llama(H.llama_config_struct(cfg, **_tiler_options(c)))
            cfg = cfg.with_(cap_bytes=H.cap_for(cfg, tg), cap_frac=0.0)
            B.tn_taskgraph_destroy(tg)
        order = None
        if c["order"] != "tiler":
            tg = B.tn_build_llama(H.llama_config_struct(cfg, **_tiler_options(c)))
            order = {"level": B.tn_taskgraph_level_order, "clustered": B.tn_taskgraph_clustered_order}[c["order"]](tg)
            B.tn_taskgraph_destroy(tg)
        self.session = H.GpuSession(cfg, _inputs(cfg, c, seed), compile_opts=H.bench_compile_opts(cfg.cap_bytes, train, pressed=c["pressed"]),
                                    n_compute=H.BENCH_COMPUTE_STREAMS, order=order, device_inputs=c["on_gpu"],
                                    device_outputs=c["on_gpu"], **_tiler_options(c))
        self.opts = B.tn_exec_opts(policy=B.TN_POLICY_BY_ORDER, max_batch=1920, queue_depth=3, max_gemm_inflight=c["gemm_inflight"],
                                   max_transfers=c["max_transfers"], copy_workgroups=c["copy_workgroups"],
                                   small_gemm_tiles=c["small_tiles"])
        # the results, tensor by tensor: the session keeps the tiles of one tensor next to each other
        s = self.session
        s.out_slab.zero_()  # the bytes between two tiles
        span = {}
        for v, off, (r, k) in zip(s.out_vids, s.out_offs, s.out_shapes):
            name, end = s.out_bind[v][1], off + r * k * cfg.elem_bytes
            lo, hi = span.get(name, (off, end))
            span[name] = (min(lo, off), max(hi, end))
        kind = torch.float32 if cfg.dtype == "f32" else torch.bfloat16
        self.results = {name: s.out_slab[lo:hi].view(kind) for name, (lo, hi) in span.items()}
        self.resident = c["on_gpu"]

    def step(self):
        if self.resident:  # device-resident inputs go to their compiled places before every execution
            self.session.place_inputs()
        self.session.execute(self.opts)
        return self.results

    def __del__(self):
        if getattr(self, "session", None) is not None:
            self.session.close()


def prepare(case, seed):
    return Program(case, seed)


def run(state):
    return state.step()


def work(case):
    c, cfg = _config(case)
    d, f, e = cfg.d_model, cfg.ffn, cfg.elem_bytes
    train = c["mode"] == "train"
    weights = cfg.layers * (4 * d * d + 3 * d * f)
    s, n = cfg.seq, cfg.decode_steps
    pairs = cfg.batch * (s * (s + 1) // 2) + n * s + n * (n + 1) // 2  # (query, key) pairs the causal mask lets through
    linear = 2.0 * cfg.tokens * weights
    attention = 4.0 * pairs * d * cfg.layers
    adapters = cfg.layers * 2.0 * cfg.tokens * LORA_RANK * 4 * d if train else 0.0
    # reverse pass: every product once for the gradient of its input (base weights are frozen), attention's scores
    # formed again and four products, the adapters' products twice
    flops = linear * (2.0 if train else 1.0) + attention * (3.5 if train else 1.0) + adapters * 3.0
    # one set of weights, shared by the layers; x in and y out; keys and values where they are outputs
    elems = weights // cfg.layers + 2 * cfg.tokens * d
    if c["kv_outputs"]:
        elems += 2 * cfg.layers * cfg.tokens * d
    if train:  # probe in, gradient of x out, adapters in and their gradients out
        elems += 2 * cfg.tokens * d + 8 * LORA_RANK * d
    return {"bytes": float(elems * e), "flops": flops}


def tolerance(case):
    """bf16: every tensor between two vertices is rounded to 8 bits, and two correct summation orders round
    differently; a layer of such tensors differs by a few 1e-3, its gradients by twice that.  fp32: the
    rounding of sums over a few thousand terms."""
    c = {**DEFAULTS, **case}
    if c["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-5}
    return {"rel": 2e-2, "max": 0.15} if c["mode"] == "train" else {"rel": 1e-2, "max": 0.1}
