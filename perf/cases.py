"""Workloads of the sparse-attention step and of the block entry, for timing them through the public entry points.

Four ways in which a program uses the framework:

  step     one denoising step over given Q / K / V tensors (FocusStep): query selection, sinks, sparse layers; replayed
           as a HIP graph, or issued call by call as a model does whose projections run between the layers
  grouped  the same step for grouped-query attention, call by call through the binding (row view of Q)
  decode   one step of a generation block (FocusDecoder): confidence from vocabulary logits, selection, cache updates,
           dense layers, probe layer, sparse layers, dense tail
  entry    the block entry (FocusDecoder): cache rewrite with block means, dense attention of every position

Keys of a case: `heads` (K/V heads), `head_dim`, `ctx` (prompt rows M), `resp` (response rows N), `gen` (positions of the
current block), `block` (prompt block size), `k` and `window` (query selection), `keep` (kept blocks), `sinks`, `layers`.
Sizes are those of the synthetic workloads (focus_inputs), of the tests, and what lies between them.
"""
from __future__ import annotations

import math

import torch

from paper_2602_02159_amd import binding as fb
from paper_2602_02159_amd.step import FocusDecoder, FocusStep

VOCAB = 126464  # rows of logits the confidence is taken from


def _case(path, heads, head_dim, ctx, resp, gen, block, k, window, keep, sinks, layers, **more):
    return dict(path=path, heads=heads, head_dim=head_dim, ctx=ctx, resp=resp, gen=gen, block=block, k=k, window=window,
                keep=keep, sinks=sinks, layers=layers, **more)


def listed():
    named = lambda name, case: dict(case, name=name)
    return [
        # the smallest step: four heads, 1K prompt; launches and latency are all there is
        named("step-1k-d64", _case("step", 4, 64, 1024, 32, 32, 64, 8, 0, 4, 2, 1, graph=True, means="cached", probe="scan")),
        # one probe scan and one sparse layer at 8K, issued call by call: the host path of a model with its own layer loop
        named("step-8k-eager", _case("step", 32, 128, 8192, 64, 64, 128, 16, 0, 6, 4, 1, graph=False, means="cached", probe="scan")),
        # a prompt and a block that divide nothing, as real prompts are
        named("step-16k-ragged", _case("step", 32, 128, 15937, 49, 49, 128, 16, 0, 6, 4, 4, graph=True, means="cached", probe="scan")),
        # the headline step: probe layer and the fifteen sparse layers of a 32-layer stack at 32K
        named("step-32k-stack", _case("step", 32, 128, 32768, 64, 64, 128, 16, 0, 7, 4, 15, graph=True, means="cached", probe="scan")),
        # the same layers for a caller that holds no block means: every layer scans K
        named("step-32k-scan", _case("step", 32, 128, 32768, 64, 64, 128, 16, 0, 7, 4, 4, graph=True, means="scan", probe="scan")),
        # the paper's hyper-parameters: nine-wide windows, half of the 64-row blocks, one sink per hundred positions
        named("step-32k-half", _case("step", 32, 128, 32768, 64, 64, 64, 4, 8, 256, 327, 4, graph=True, means="cached", probe="scan")),
        # the longest context
        named("step-128k", _case("step", 32, 128, 131072, 64, 64, 128, 16, 0, 30, 4, 2, graph=True, means="cached", probe="scan")),
        # 28 query heads on 4 K/V heads, window-expanded queries, sinks from the probe layer's own attention
        named("grouped-16k", _case("grouped", 4, 128, 16384, 256, 32, 64, 4, 8, 128, 163, 4, group=7)),
        # a decoding step as the paper lays it out: 256 response rows, a 32-position block, logits in, dense and sparse layers
        named("decode-32k", _case("decode", 32, 128, 32768, 256, 32, 64, 4, 8, 256, 327, 8, l_dense=3, tail=1, logits=True)),
        # block entries: a few short rows, an ordinary prompt, the longest one
        named("entry-1k-d64", _case("entry", 4, 64, 1024, 32, 32, 64, 8, 0, 4, 2, 2)),
        named("entry-8k", _case("entry", 32, 128, 8192, 64, 64, 128, 16, 0, 6, 4, 2)),
        named("entry-32k", _case("entry", 32, 128, 32768, 64, 64, 128, 16, 0, 7, 4, 1)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: contexts of 1000 to 131072 rows (block entries: to 32768), any length in between."""
    path = rng.choice(("step", "step", "step", "grouped", "decode", "entry", "entry"))
    head_dim = rng.choice((64, 128, 128, 128))
    heads = rng.choice((2, 4, 8)) if path == "grouped" else rng.choice((4, 8, 16, 32, 32))
    ctx = _log_int(rng, 1000, 32768 if path in ("entry", "decode") else 131072)
    block = rng.choice((64, 128))
    gen = rng.randint(32, 64)
    resp = gen if rng.random() < 0.5 else rng.randint(gen, 256)
    k, window = rng.choice(((4, 8), (8, 2), (8, 0), (16, 0), (16, 0)))
    n_b = -(-ctx // block)
    keep = min(n_b, max(2, int(n_b * math.exp(rng.uniform(math.log(0.03), math.log(0.5))))))
    sinks = max(2, ctx // 100) if rng.random() < 0.4 else rng.choice((2, 4, 16))
    c = _case(path, heads, head_dim, ctx, resp, gen, block, k, window, keep, sinks, 1)
    rows = heads * head_dim * (ctx + resp) * 4  # bytes of one layer's K and V
    if path == "step":
        c["layers"] = max(1, min(rng.choice((1, 2, 4, 8)), int(8e9 // rows)))
        c.update(graph=rng.random() < 0.7, means=rng.choice(("cached", "cached", "cached", "scan")), probe=rng.choice(("scan", "scan", "layer")))
    elif path == "grouped":
        c.update(layers=rng.randint(1, 4), group=rng.choice((4, 7, 8)))
    elif path == "decode":
        c.update(layers=rng.randint(4, 8), l_dense=rng.randint(0, 1), tail=rng.randint(0, 1), logits=rng.random() < 0.5)
    else:
        c["layers"] = rng.randint(1, 2) if ctx < 16384 else 1
    return c


# ---- inputs: normal Q, K, V; a few keys with a shared direction that every query also has a share of (attention sinks)
class _Inputs:
    def __init__(self, case, seed):
        self.dev = torch.device("cuda")
        self.g = torch.Generator(device=self.dev).manual_seed(seed)
        self.case = case
        d = case["head_dim"]
        u = self.normal(d, dtype=torch.float32)
        self.u = u / torch.linalg.vector_norm(u)
        gain = math.sqrt(6.0 * math.sqrt(d) / 2.0)  # a sink's logit exceeds the others by six
        self.q_dir, self.k_dir = 0.5 * gain * self.u, 4.0 * gain * self.u
        self.sink_rows = torch.randint(0, case["ctx"], (4,), generator=self.g, device=self.dev)

    def normal(self, *shape, dtype=torch.bfloat16):
        return torch.randn(shape, generator=self.g, device=self.dev, dtype=dtype)

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.g, device=self.dev)

    def fill_q(self, t):
        t.normal_(generator=self.g).add_(self.q_dir.to(t.dtype))

    def fill_k(self, t):
        t.normal_(generator=self.g)
        t[:, self.sink_rows] += self.k_dir.to(t.dtype)

    def fill_v(self, t):
        t.normal_(generator=self.g)

    def qkv(self, q_rows, rows):
        H, d = self.case["heads"], self.case["head_dim"]
        q, k, v = (torch.empty((H, n, d), dtype=torch.bfloat16, device=self.dev) for n in (q_rows, rows, rows))
        self.fill_q(q)
        self.fill_k(k)
        self.fill_v(v)
        return q, k, v

    def confidence(self):
        gen = self.case["gen"]
        return 0.8 * self.uniform(gen) + 0.2 * self.uniform(gen)

    def masked(self):
        """A quarter of the block is unmasked already."""
        gen = self.case["gen"]
        m = torch.ones(gen, dtype=torch.uint8, device=self.dev)
        m[torch.randperm(gen, generator=self.g, device=self.dev)[:gen // 4]] = 0
        return m

    def logits(self):
        gen = self.case["gen"]
        t = self.normal(gen, VOCAB).mul_(3.0)
        peak = torch.randint(0, VOCAB, (gen,), generator=self.g, device=self.dev)
        t[torch.arange(gen, device=self.dev), peak] += (8.0 + 12.0 * self.uniform(gen)).to(t.dtype)
        return t


def _prepare_step(case, x):
    rows = case["ctx"] + case["resp"]
    probe = x.qkv(case["gen"], rows)
    if case["probe"] == "scan":
        probe = probe[:2]
    layers = [x.qkv(case["gen"], rows) for _ in range(case["layers"])]
    step = FocusStep(x.confidence(), x.masked(), probe, layers, case["ctx"], case["block"], case["k"], case["window"], case["keep"],
                     case["sinks"], cached_means=case["means"] == "cached")
    step.use_probe_layer = case["probe"] == "layer"
    if case["means"] == "cached":
        step.issue("block_means")  # what the block entry leaves behind
    if case["graph"]:
        step.capture()
    outputs = {"focus": step.focus_idx, "active": step.active_idx, "counts": step.counts, "sinks": step.sink_idx,
               "col_mass": step.col_mass, "layers": [{n: b[n] for n in ("kept", "scores", "out")} for b in step.bufs]}
    if step.use_probe_layer:
        outputs["probe_out"] = step.probe_out
    return step.run, outputs


def _prepare_grouped(case, x):
    dev, H, d, group = x.dev, case["heads"], case["head_dim"], case["group"]
    M, B, gen, k = case["ctx"], case["block"], case["gen"], case["k"]
    cap = min(gen, k * (2 * (case["window"] // 2) + 1))
    i32 = lambda n: torch.full((n,), -1, dtype=torch.int32, device=dev)
    conf, masked = x.confidence(), x.masked()
    focus, active, counts = i32(k), i32(cap), i32(2)
    g_focus, g_active, g_counts, sinks = i32(group * k), i32(group * cap), i32(2), i32(case["sinks"])
    col_mass = torch.zeros(M + case["resp"], device=dev)
    n_b = -(-M // B)
    layers = []
    for l in range(case["layers"] + 1):  # the probe layer, then the sparse ones
        q, kk, v = x.qkv(group * gen, M + case["resp"])
        out = torch.zeros((H, group * cap, d), dtype=torch.bfloat16, device=dev)
        shape = fb.make_shape(q, kk, v, M, B, out)
        fn = fb.FN_SPARSE_LAYER if l else fb.FN_PROBE_LAYER
        ws = torch.empty(fb.workspace_bytes(fn, shape, group * cap, case["keep"], case["sinks"]), dtype=torch.uint8, device=dev)
        kbar = torch.zeros((H, n_b, d), device=dev)
        fb.block_means(kk, shape, kbar)
        layers.append((q, kk, v, kbar, shape, torch.zeros(n_b, device=dev), i32(case["keep"]), out, ws))

    def step():
        fb.select_queries(conf, masked, k, case["window"], 0, gen, focus, active, counts)
        fb.expand_groups(focus, active, counts, gen, group, g_focus, g_active, g_counts)
        q, kk, v, _, shape, _, _, out, ws = layers[0]
        fb.probe_layer(q, g_active, g_counts, kk, v, shape, case["sinks"], out, None, col_mass, sinks, ws)
        for q, kk, v, kbar, shape, scores, kept, out, ws in layers[1:]:
            fb.sparse_layer(q, g_focus, g_active, g_counts, kk, v, kbar, shape, case["keep"], sinks, case["sinks"], scores, kept,
                            out, None, ws)

    outputs = {"focus": g_focus, "active": g_active, "counts": g_counts, "sinks": sinks, "col_mass": col_mass, "probe_out": layers[0][7],
               "layers": [{"scores": t[5], "kept": t[6], "out": t[7]} for t in layers[1:]]}
    return step, outputs


def _decoder(case, x):
    dec = FocusDecoder(case["layers"], case.get("l_dense", 0), case.get("tail", 0), case["heads"], case["head_dim"], case["ctx"], case["resp"],
                       case["gen"], case["ctx"], case["block"], case["k"], case["window"], case["keep"], case["sinks"], x.dev,
                       VOCAB if case.get("logits") else None)
    for l in range(case["layers"]):
        x.fill_q(dec.q_all[l])
        x.fill_k(dec.k_all[l])
        x.fill_v(dec.v_all[l])
        x.fill_q(dec.q[l])
        x.fill_v(dec.k_new[l])
        x.fill_v(dec.v_new[l])
    dec.conf.copy_(x.confidence())
    dec.masked.copy_(x.masked())
    if dec.logits is not None:
        dec.logits.copy_(x.logits())
    dec.capture()
    return dec


def _prepare_decode(case, x):
    dec = _decoder(case, x)
    dec.run_entry()
    sparse = [l for l in range(case["layers"]) if dec.is_sparse(l)]
    outputs = {"tokens": dec.tokens, "conf": dec.conf, "focus": dec.focus_idx, "active": dec.active_idx, "counts": dec.counts,
               "sinks": dec.sink_idx, "col_mass": dec.col_mass, "out": dec.out, "k_cache": dec.k_cache, "v_cache": dec.v_cache,
               "kept": [dec.kept[l] for l in sparse], "scores": [dec.scores[l] for l in sparse]}
    return dec.run_step, outputs


def _prepare_entry(case, x):
    dec = _decoder(case, x)
    outputs = {"out": dec.out_all, "k_cache": dec.k_cache, "v_cache": dec.v_cache, "kbar": [t for t in dec.kbar if t is not None]}
    return dec.run_entry, outputs


def prepare(case, seed):
    x = _Inputs(case, seed)
    return {"step": _prepare_step, "grouped": _prepare_grouped, "decode": _prepare_decode, "entry": _prepare_entry}[case["path"]](case, x)


def run(state):
    go, outputs = state
    go()
    return outputs


def _active(case):
    """Expected size of the union of the k windows."""
    span, gen = 2 * (case["window"] // 2) + 1, case["gen"]
    return case["k"] if span == 1 else gen * (1.0 - (1.0 - min(1.0, span / gen)) ** case["k"])


def work(case):
    H, d, M, L = case["heads"], case["head_dim"], case["ctx"], case["ctx"] + case["resp"]
    n_b = -(-M // case["block"])
    row = H * d * 2  # bytes of one position over all K/V heads
    if case["path"] == "entry":
        n_sparse = case["layers"] - 1  # the first layer is the probe: it keeps no block means
        return {"bytes": case["layers"] * 6 * L * row + n_sparse * n_b * H * d * 4, "flops": case["layers"] * 4.0 * L * L * H * d}
    n_q = _active(case) * case.get("group", 1)
    kept = min(M, case["keep"] * case["block"])
    keys = kept + case["resp"] + case["sinks"] * (1.0 - kept / M)
    q_out = 2 * n_q * row
    scan = case.get("means") == "scan"
    sparse = {"bytes": 2 * keys * row + q_out + ((M - kept) * row if scan else n_b * H * d * 4), "flops": 4.0 * n_q * keys * H * d}
    dense = {"bytes": 2 * L * row + q_out, "flops": 4.0 * n_q * L * H * d}
    probe = {"bytes": dense["bytes"] + 4 * L, "flops": dense["flops"]}
    if case.get("probe") == "scan":
        probe = {"bytes": (L + n_q) * row + 4 * L, "flops": 2.0 * n_q * L * H * d}
    if case["path"] == "decode":
        n_dense = case["l_dense"] + case["tail"]
        parts = [(1, probe), (n_dense, dense), (case["layers"] - n_dense - 1, sparse), (case["layers"], {"bytes": 4 * n_q * row, "flops": 0.0})]
        parts.append((1, {"bytes": case["gen"] * VOCAB * 2 if case["logits"] else 0, "flops": 0.0}))
    else:
        parts = [(1, probe), (case["layers"], sparse)]
    return {key: sum(n * p[key] for n, p in parts) + (5 * case["gen"] if key == "bytes" else 0) for key in ("bytes", "flops")}


def tolerance(case):
    """Attention outputs are bf16 with bf16 probabilities; scores and masses are fp32 sums; two of the many column masses or
    scores may be so close that fp32 rounding orders them."""
    return {"rel": 1e-2, "max": 0.1, "differ": 0.005}
