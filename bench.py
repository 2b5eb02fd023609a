"""Benchmark: decode latency of compiled structured-sparse plans vs the dense plan on one MI355X.

Workload (default, `llama3_70b_stack`): the full 80-layer Llama-3-70B-shaped decode step at batch
1 (hidden 8192, 64 / 8 heads, head_dim 128, SwiGLU 28672, INT8 per-row weights, 4096 prior
positions in the BF16 cache, final RMSNorm and the dense 128256 x 8192 BF16 LM head), the seed-1
43%-reduction mask against the dense plan. A step is one token through every layer and the LM
head, replayed from a HIP graph (how a serving loop issues a fixed plan). `value` is the mean of
five timing blocks of 200 steps (each after 50 warm-up steps), as the paper times its decode.

Output: one JSON line with the metric, the dense comparison, the achieved HBM bandwidth, the
roofline of the dominant kernel (the gate/up GEMVs of all layers, timed per launch with HIP events
on the launch stream), the measured HBM traffic of that kernel where a counter summary of the
current kernel source exists, the CPU oracle timed on the host cores as a baseline, a run manifest,
and (default workload only) the one-layer and 32-layer Llama-3-8B-shaped numbers as extras.
Other workloads: `--workload` (see synth.WORKLOADS).
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "ms/token decode at batch 1 (sparse vs dense) + achieved HBM GB/s % of peak"
PEAK_GBPS = 8000.0
STAGE_KIND = {"attention": 1, "gateup_gemv": 3}
ROTATE_BYTES = 2.5e9


def parse():
    p = argparse.ArgumentParser()
    p.add_argument("--gpus", type=int, default=1)
    p.add_argument("--steps", type=int, default=1000)
    p.add_argument("--warmup", type=int, default=50)
    p.add_argument("--workload", default="llama3_70b_stack")
    p.add_argument("--mask-seed", type=int, default=1)
    p.add_argument("--blocks", type=int, default=5)
    p.add_argument("--timed-launches", type=int, default=64)
    p.add_argument("--cpu-seconds", type=float, default=12.0)
    p.add_argument("--no-cpu", action="store_true")
    p.add_argument("--no-extras", action="store_true",
                   help="default workload: skip the 8B layer and 8B stack extras")
    p.add_argument("--block-warmup", type=int, default=50)
    p.add_argument("--block-steps", type=int, default=200)
    p.add_argument("--sparse-only", action="store_true",
                   help="time only the sparse plan (counter runs); no JSON metric line")
    return p.parse_args()


def source_hash(files):
    h = hashlib.sha256()
    for f in files:
        with open(os.path.join(ROOT, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def layer_bytes(sh, m_q, m_kv, c, pos, batch=1):
    """Algorithmic HBM bytes of one decode step of one layer and of its gate/up GEMV."""
    d, dh = sh.d_model, sh.head_dim
    w = (m_q + 2 * m_kv) * dh * d + d * m_q * dh + 3 * d * c
    s = 4 * ((m_q + 2 * m_kv) * dh + d + 2 * c + d)
    kv = batch * m_kv * (pos + 1) * dh * 2 * 2
    gateup = 2 * c * d + 2 * c * 4 + batch * (d * 4 + c * 4)
    # split-KV attention with its merge: cache rows, q/k/v in, new k/v rows written, o out
    attention = kv + batch * ((m_q + 2 * m_kv) * dh * 4 + 2 * m_kv * dh * 2 + m_q * dh * 4)
    return {"weights": w, "scales": s, "kv": kv, "total": w + s + kv, "gateup": gateup,
            "attention": attention}


def stack_bytes(sh, counts, pos):
    """Algorithmic HBM bytes of one batch-1 decode step of a stack: every layer's retained INT8
    weights, row scales and retained KV rows (per-layer counts (m_q, m_kv, c)), plus the BF16 LM
    head (2 V d bytes)."""
    tot = {"weights": 0, "scales": 0, "kv": 0}
    for m_q, m_kv, c in counts:
        nb = layer_bytes(sh, m_q, m_kv, c, pos, 1)
        for k in tot:
            tot[k] += nb[k]
    tot["lm_head"] = 2 * sh.vocab * sh.d_model
    tot["total"] = tot["weights"] + tot["scales"] + tot["kv"] + tot["lm_head"]
    return tot


def dense_layer_flops(sh):
    """Active FLOPs per token of the full-width stack: per layer 2 d d_h (H_q + 2 H_kv) for QKV,
    2 d_h H_q d for O and 6 d F for gate, up and down."""
    d, dh = sh.d_model, sh.head_dim
    return sh.n_layers * (2 * d * dh * (sh.n_q_heads + 2 * sh.n_kv_heads)
                          + 2 * dh * sh.n_q_heads * d + 6 * d * sh.d_ffn)


class Rotation:
    """R compiled copies of one plan with their own KV caches, and HIP graphs of one step each."""

    def __init__(self, S, torch, sh, desc, dstore, mask, prior, x, pos, copies, make_plan=None):
        """make_plan(i): the plan of copy i (default: a plan of `mask` compiled from dstore)."""
        self.plans, self.caches = [], []
        batch = x.shape[0]
        self.batch = batch
        for i in range(copies):
            plan = make_plan(i) if make_plan else S.Plan(desc, dstore, mask)
            cache = S.KVCache(desc, batch, pos + 1)
            cache.load_layer(0, *prior)
            plan.bind(cache)
            self.plans.append(plan)
            self.caches.append(cache)
        self.torch, self.pos = torch, pos
        self.x = torch.from_numpy(x).cuda()
        self.out = torch.empty_like(self.x)
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        st = torch.cuda.Stream()
        st.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(st):           # warm the launch path before capture
            self.step_all(S.current_stream())
        torch.cuda.current_stream().wait_stream(st)
        torch.cuda.synchronize()
        with torch.cuda.graph(self.graph):
            self.step_all(S.current_stream())
        torch.cuda.synchronize()
        self.S = S

    def step_all(self, stream):
        for plan, cache in zip(self.plans, self.caches):
            plan.decode(self.x, cache, self.pos, self.out, stream=stream)

    def run_steps(self, n):
        """Issue n decode steps: whole-graph replays plus single eager steps for the remainder."""
        R = len(self.plans)
        for _ in range(n // R):
            self.graph.replay()
        for i in range(n % R):
            self.plans[i].decode(self.x, self.caches[i], self.pos, self.out)

    def time_eager(self, n):
        """Mean step time (ms) of n decode steps issued as plain launches (no graph)."""
        torch = self.torch
        R = len(self.plans)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for i in range(n):
            self.plans[i % R].decode(self.x, self.caches[i % R], self.pos, self.out)
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / n

    def time_steps(self, n):
        torch = self.torch
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        self.run_steps(n)
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / n

    def stage_ms(self, kind, reps=20):
        """Mean duration (ms) of one stage kernel over back-to-back launches across the copies."""
        return self.S.B.tasp_profile_stage([p.handle for p in self.plans],
                                           [c.struct for c in self.caches], 0, kind, self.pos,
                                           reps, self.S.current_stream())

    def kernel_times(self, launches):
        """Per-kernel durations (ms) from HIP events around each launch, over the copies."""
        acc = {}
        R = len(self.plans)
        for i in range(launches):
            for name, ms in self.plans[i % R].decode_timed(self.x, self.caches[i % R], self.pos, self.out):
                acc.setdefault(name, []).append(ms)
        return {k: float(np.mean(v)) for k, v in acc.items()}


def cpu_baseline(sh, store_layer, mask, prior, x, pos, budget_s):
    import threadpoolctl
    from oracle import reference as ref
    closed = ref.close_mask(*(mask if mask is not None else
                              (np.ones((1, sh.n_q_heads), np.uint8), None, np.ones((1, sh.d_ffn), np.uint8))),
                            sh.group_size)
    W = ref.masked_layer(store_layer, closed[0][0], closed[1][0], closed[2][0], sh.head_dim)
    K = prior[0].astype(np.uint32) << 16
    V = prior[1].astype(np.uint32) << 16
    K = K.view(np.float32).astype(np.float64)
    V = V.view(np.float32).astype(np.float64)
    ref.decode_layer(W, x, K.copy(), V.copy(), pos, sh)          # warm-up
    times = []
    t_start = time.perf_counter()
    while time.perf_counter() - t_start < budget_s or len(times) < 3:
        t0 = time.perf_counter()
        ref.decode_layer(W, x, K, V, pos, sh)
        times.append(time.perf_counter() - t0)
    info = threadpoolctl.threadpool_info()
    threads = max([i.get("num_threads", 1) for i in info] or [1])
    return {"value": float(np.median(times) * 1e3), "unit": "ms/token", "cores": int(threads),
            "kind": "oracle",
            "sample": f"{len(times)} oracle decode steps of the same layer (float64 numpy, "
                      f"zero-masked dequantised weights resident; dequantisation excluded), median",
            "host_cpus": len(os.sched_getaffinity(0))}


def copy_probe_gbps(torch, B, nbytes=1 << 30, reps=10):
    """Read + write bandwidth of the library's plain streaming copy over 1 GiB buffers."""
    src = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    dst = torch.empty_like(src)
    stream = torch.cuda.current_stream().cuda_stream
    for _ in range(2):
        B.tasp_copy_probe(dst.data_ptr(), src.data_ptr(), nbytes, stream)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        B.tasp_copy_probe(dst.data_ptr(), src.data_ptr(), nbytes, stream)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / reps
    del src, dst
    torch.cuda.empty_cache()
    return 2 * nbytes / (ms * 1e-3) / 1e9


def device_layer(torch, sh, gen):
    """One decoder layer of the INT8 store drawn on the GPU: N(0, 0.02) rows quantised to INT8 with
    one float32 scale per row (max |w| / 127), BF16(1 + 0.1 N(0, 1)) gains. Used for stacks, whose
    stores (5-70 GB) are too large to draw on the host."""
    qd, kd, d, f = sh.n_q_heads * sh.head_dim, sh.n_kv_heads * sh.head_dim, sh.d_model, sh.d_ffn
    out = {}
    for name, (rows, cols) in (("wq", (qd, d)), ("wk", (kd, d)), ("wv", (kd, d)), ("wo", (d, qd)),
                               ("wg", (f, d)), ("wu", (f, d)), ("wd", (d, f))):
        w = torch.randn(rows, cols, generator=gen, device="cuda") * 0.02
        s = (w.abs().amax(dim=1) / 127.0).clamp_min(1e-30)
        q = torch.round(w / s[:, None]).clamp_(-127, 127).to(torch.int8)
        out[name] = (q, s.float().contiguous())
        del w
    for name in ("attn_norm", "ffn_norm"):
        g = (1.0 + 0.1 * torch.randn(d, generator=gen, device="cuda")).to(torch.bfloat16)
        out[name] = g.view(torch.int16)
    return out


def device_group_layer(torch, sh, gen):
    """One decoder layer of the groupwise store drawn on the GPU: N(0, 0.02) weights quantised to
    INT8 with one BF16 scale per row and 128 inputs (max |w| of the group / 127, rounded to BF16
    before quantising), BF16(1 + 0.1 N(0, 1)) gains; scales as int16 bit patterns."""
    qd, kd, d, f = sh.n_q_heads * sh.head_dim, sh.n_kv_heads * sh.head_dim, sh.d_model, sh.d_ffn
    out = {}
    for name, (rows, cols) in (("wq", (qd, d)), ("wk", (kd, d)), ("wv", (kd, d)), ("wo", (d, qd)),
                               ("wg", (f, d)), ("wu", (f, d)), ("wd", (d, f))):
        w = (torch.randn(rows, cols, generator=gen, device="cuda") * 0.02).view(rows, cols // 128, 128)
        s = (w.abs().amax(dim=2) / 127.0).clamp_min(1e-30).to(torch.bfloat16)
        q = torch.round(w / s.float()[:, :, None]).clamp_(-127, 127).to(torch.int8).view(rows, cols)
        out[name] = (q, s.view(torch.int16).contiguous())
        del w
    for name in ("attn_norm", "ffn_norm"):
        g = (1.0 + 0.1 * torch.randn(d, generator=gen, device="cuda")).to(torch.bfloat16)
        out[name] = g.view(torch.int16)
    return out


def bench_shared_stack(args, wl):
    """Batch-1 decode of a full stack from one shared groupwise store: every plan (the seed mask,
    then the dense plan) indexes the same store through its maps and owns no weight bytes. Per
    plan: args.warmup graph replays, args.steps timed, then args.blocks blocks of
    args.block_warmup + args.block_steps replays."""
    import torch
    import synth
    from paper_2609_29499_amd import binding as B
    from paper_2609_29499_amd import session as S
    sh, pos = wl.shape, wl.pos
    gen = torch.Generator(device="cuda")
    gen.manual_seed(0)
    t0 = time.time()
    layers = [device_group_layer(torch, sh, gen) for _ in range(sh.n_layers)]
    fnorm = (1.0 + 0.1 * torch.randn(sh.d_model, generator=gen, device="cuda")).to(torch.bfloat16).view(torch.int16)
    lm = (0.02 * torch.randn(sh.vocab, sh.d_model, generator=gen, device="cuda")).to(torch.bfloat16).view(torch.int16)
    store = S.GroupStore(layers, fnorm, lm)
    del layers
    desc = S.desc_from_shape(sh, max_batch=1, max_seq=pos + 1)
    torch.cuda.synchronize()
    print(f"[bench] {wl.name}: store {store.nbytes() / 1e9:.1f} GB drawn in {time.time() - t0:.1f}s",
          file=sys.stderr, flush=True)
    x = torch.randn(1, sh.d_model, generator=gen, device="cuda").to(torch.bfloat16).float()
    out = torch.empty(1, sh.vocab, device="cuda")
    scratch = S.SharedScratch(desc)
    plans = [(f"mask{sd}", synth.budget_mask(sh, sd)) for sd in wl.mask_seeds] + [("dense", None)]
    rows = []
    for name, m in plans:
        plan = S.Plan.shared(desc, store, m, scratch=scratch)
        cache = S.KVCache(desc, 1, pos + 1)
        for l in range(sh.n_layers):
            cache.k[l, :, :, :pos].normal_(generator=gen)
            cache.v[l, :, :, :pos].normal_(generator=gen)
        plan.bind(cache)
        for _ in range(3):
            plan.decode(x, cache, pos, out)
        torch.cuda.synchronize()
        g = _graph_of(torch, S, plan, x, cache, pos, out)
        for _ in range(args.warmup):
            g.replay()
        ms = _time_replays(torch, g, args.steps)
        blocks = []
        for _ in range(args.blocks):
            for _ in range(args.block_warmup):
                g.replay()
            blocks.append(_time_replays(torch, g, args.block_steps))
        bmean = float(np.mean(blocks)) if blocks else ms
        rows.append({"plan": name, "ms_per_token": round(bmean, 5), "ms_per_step": round(ms, 5),
                     "blocks_ms": [round(b, 5) for b in blocks],
                     "plan_workspace_MB": round(plan.ws_bytes / 1e6, 3),
                     "active_flop_ratio": round(plan.ledger()["active_flop_ratio"], 4)})
        print(f"[bench] {name}: {bmean:.4f} ms/token (blocks), {ms:.4f} (timed steps)",
              file=sys.stderr, flush=True)
        del cache, g, plan
        torch.cuda.empty_cache()
    sp, dn = rows[0], rows[-1]
    line = {
        "metric": METRIC, "value": sp["ms_per_token"], "unit": "ms/token", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": sp["ms_per_step"],
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "int8w-g128-f32",
        "data": "synthetic",
        "config": {"workload": wl.name, "d_model": sh.d_model, "layers": sh.n_layers, "batch": 1,
                   "pos": pos, "mask_seed": wl.mask_seeds[0], "vocab": sh.vocab,
                   "scales": "BF16 per 128 inputs"},
        "dense_ms_per_token": dn["ms_per_token"],
        "speedup_vs_dense": round(dn["ms_per_token"] / sp["ms_per_token"], 4),
        "plans": rows,
        "memory_GB": {"store_with_scales_gains_and_lm_head": round(store.nbytes() / 1e9, 2),
                      "shared_scratch": round(scratch.bytes / 1e9, 3)},
        "roofline": None, "cpu_baseline": None,
        "paper_context": "one packed store serves every mask; a mask owns no weight bytes (appendix "
                         "'Backing-store semantics')",
        "manifest": run_manifest(),
    }
    print(json.dumps(line), flush=True)


def _graph_of(torch, S, plan, x, cache, pos, out):
    """A HIP graph holding one decode step of `plan` (captured on a side stream after a warm
    launch)."""
    g = torch.cuda.CUDAGraph()
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(st):
        plan.decode(x, cache, pos, out, stream=S.current_stream())
    torch.cuda.current_stream().wait_stream(st)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        plan.decode(x, cache, pos, out, stream=S.current_stream())
    torch.cuda.synchronize()
    return g


def _time_replays(torch, g, n):
    """Mean ms per replay of n back-to-back replays between two events."""
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(n):
        g.replay()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / n


def measure_stack(args, sh, pos, mask_seeds, timed_steps=5):
    """ms/token of a full decode step (all layers + final norm + BF16 LM head) for every seeded
    mask and then the dense plan, batch 1, cache at pos prior positions: one row per plan, in
    that order (sparse first, so a kernel trace splits at the first dense-shaped launch).

    Per plan: args.warmup replays, then args.steps timed replays (ms_per_step), then args.blocks
    blocks of args.block_warmup + args.block_steps replays (the paper's protocol); per-kernel HIP
    events over `timed_steps` eager steps give the gate/up GEMV and LM head durations."""
    import torch
    import synth
    from paper_2609_29499_amd import session as S
    gen = torch.Generator(device="cuda")
    gen.manual_seed(0)
    t0 = time.time()
    layers = [device_layer(torch, sh, gen) for _ in range(sh.n_layers)]
    fnorm = (1.0 + 0.1 * torch.randn(sh.d_model, generator=gen, device="cuda")).to(torch.bfloat16).view(torch.int16)
    lm = (0.02 * torch.randn(sh.vocab, sh.d_model, generator=gen, device="cuda")).to(torch.bfloat16).view(torch.int16)
    store = S.DeviceStore(layers, fnorm, lm)
    desc = S.desc_from_shape(sh, max_batch=1, max_seq=pos + 1)
    torch.cuda.synchronize()
    print(f"[bench] stack: store drawn in {time.time() - t0:.1f}s", file=sys.stderr, flush=True)
    plans = [(f"mask{sd}", synth.budget_mask(sh, sd)) for sd in mask_seeds]
    if args.sparse_only:        # counter runs: the first mask alone
        plans = plans[:1]
    else:
        plans.append(("dense", None))
    x = torch.randn(1, sh.d_model, generator=gen, device="cuda").to(torch.bfloat16).float()
    out = torch.empty(1, sh.vocab, device="cuda")
    rows = []
    # one plan at a time: the store plus the largest plan (the dense copy) bound device memory
    for name, m in plans:
        plan = S.Plan(desc, store, m)
        cache = S.KVCache(desc, 1, pos + 1)
        for l in range(sh.n_layers):
            cache.k[l, :, :, :pos].normal_(generator=gen)
            cache.v[l, :, :, :pos].normal_(generator=gen)
        plan.bind(cache)
        for _ in range(3):
            plan.decode(x, cache, pos, out)
        torch.cuda.synchronize()
        g = _graph_of(torch, S, plan, x, cache, pos, out)
        for _ in range(args.warmup):
            g.replay()
        ms = _time_replays(torch, g, args.steps)
        blocks = []
        for _ in range(args.blocks):
            for _ in range(args.block_warmup):
                g.replay()
            blocks.append(_time_replays(torch, g, args.block_steps))
        # LM head: HIP events around each kernel of eager steps on the launch stream; gate/up:
        # back-to-back launches of every layer's gate/up GEMV between two HIP events on the launch
        # stream (each launch reads another layer's panel, as in a step)
        lm_ms = []
        for _ in range(timed_steps):
            kt = plan.decode_timed(x, cache, pos, out)
            lm_ms.append(sum(t for k, t in kt if k == "lmhead_gemv"))
        lm_ms = float(np.median(lm_ms))
        gu_reps = 2
        gu_launch_ms = S.B.tasp_profile_stage([plan.handle], [cache.struct], -1, STAGE_KIND["gateup_gemv"],
                                              pos, gu_reps, S.current_stream())
        gu_launch = [gu_launch_ms] * (gu_reps * sum(1 for l in range(sh.n_layers) if plan.counts(l)[2] > 0))
        counts = [plan.counts(l) for l in range(sh.n_layers)]
        d = sh.d_model
        gu_bytes = sum(2 * c * d + 2 * c * 4 + d * 4 + c * 4 for _, _, c in counts)
        nb = stack_bytes(sh, counts, pos)
        led = plan.ledger()
        bmean = float(np.mean(blocks)) if blocks else ms
        rows.append({"plan": name, "ms_per_token": round(bmean, 5), "ms_per_step": round(ms, 5),
                     "blocks_ms": [round(b, 5) for b in blocks],
                     "blocks_mean_sd_ms": [round(bmean, 5),
                                           round(float(np.std(blocks, ddof=1)), 5) if len(blocks) > 1 else 0.0],
                     "us_per_layer": round((bmean - lm_ms) * 1e3 / sh.n_layers, 3),
                     "lm_head_ms": round(lm_ms, 5),
                     "gateup_avg_launch_us": round(float(np.mean(gu_launch)) * 1e3, 3),
                     "gateup_launches_timed": len(gu_launch),
                     "gateup_bytes_per_launch": round(gu_bytes / sh.n_layers),
                     "bytes": nb["total"], "kv_bytes": nb["kv"], "lm_head_bytes": nb["lm_head"],
                     "GBps": round(nb["total"] / (bmean * 1e-3) / 1e9, 1),
                     "active_flop_ratio": round(led["active_flop_ratio"], 4)})
        print(f"[bench] {name}: {bmean:.4f} ms/token (blocks), {ms:.4f} (timed steps), "
              f"{rows[-1]['GBps']} GB/s, gate/up {rows[-1]['gateup_avg_launch_us']} us/launch",
              file=sys.stderr, flush=True)
        del cache, g, plan
        torch.cuda.empty_cache()
    del store, layers
    torch.cuda.empty_cache()
    return rows


def host_cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for ln in f:
                if ln.startswith("model name"):
                    return ln.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


SOURCE_FILES = ["bench.py", "include/tasp.h", "paper_2609_29499_amd/session.py",
                "paper_2609_29499_amd/binding.py"]


def run_manifest():
    """What ran where: the commit (when the tree is a git checkout) and a hash of the library and
    bench sources, ROCm / torch / HIP versions, the GPU and the host CPU."""
    import subprocess
    import torch
    man = {}
    try:
        r = subprocess.run(["git", "rev-parse", "HEAD"], cwd=ROOT, capture_output=True, text=True,
                           timeout=10)
        man["git_sha"] = r.stdout.strip() or None
    except (OSError, subprocess.SubprocessError):
        man["git_sha"] = None
    csrc = os.path.join(ROOT, "paper_2609_29499_amd", "csrc")
    files = SOURCE_FILES + sorted(os.path.join("paper_2609_29499_amd", "csrc", f)
                                  for f in os.listdir(csrc))
    man["source_sha"] = source_hash(files)
    try:
        with open("/opt/rocm/.info/version") as f:
            man["rocm"] = f.read().strip()
    except OSError:
        man["rocm"] = None
    man["torch"] = torch.__version__
    man["hip_runtime"] = getattr(torch.version, "hip", None)
    props = torch.cuda.get_device_properties(0)
    man["gpu"] = props.name
    man["gpu_arch"] = getattr(props, "gcnArchName", None)
    man["host_cpu"] = host_cpu_model()
    man["host_cpus"] = len(os.sched_getaffinity(0))
    return man


def stack_line(args, wl, rows):
    """The JSON line of a stack workload from measure_stack's rows."""
    sh, pos = wl.shape, wl.pos
    sparse = [r for r in rows if r["plan"] != "dense"]
    dense = next((r for r in rows if r["plan"] == "dense"), None)
    mean_sparse = float(np.mean([r["ms_per_token"] for r in sparse]))
    ms_steps = float(np.mean([r["ms_per_step"] for r in sparse]))
    sp0 = sparse[0]
    gu_gbps = sp0["gateup_bytes_per_launch"] / (sp0["gateup_avg_launch_us"] * 1e-6) / 1e9
    line = {
        "metric": METRIC, "value": round(mean_sparse, 5), "unit": "ms/token", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms_steps, 5),
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "int8w-f32",
        "data": "synthetic",
        "config": {"workload": wl.name, "d_model": sh.d_model, "n_q_heads": sh.n_q_heads,
                   "n_kv_heads": sh.n_kv_heads, "head_dim": sh.head_dim, "d_ffn": sh.d_ffn,
                   "layers": sh.n_layers, "vocab": sh.vocab, "batch": 1, "pos": pos,
                   "masks": list(wl.mask_seeds)},
        "value_protocol": f"mean of {args.blocks} blocks x {args.block_steps} graph replays "
                          f"(each after {args.block_warmup} warm-up replays) over the sparse plans",
        "plans": rows,
        "achieved_GBps": round(float(np.mean([r["GBps"] for r in sparse])), 1),
        "hbm_frac": round(float(np.mean([r["GBps"] for r in sparse])) / PEAK_GBPS, 4),
        "us_per_layer": round(float(np.mean([r["us_per_layer"] for r in sparse])), 3),
        "paper_context": "45.2 -> 31.3 ms/token dense vs compiled sparse, Llama-3-70B, INT8/BF16, one A100 80GB",
        # the kernel that moves the most bytes of the step: the gate/up GEMVs (one per layer),
        # per-launch HIP events on the launch stream in eager steps of the first masked plan
        "roofline": {"bound": "hbm", "kernel": "gateup_gemv",
                     "achieved": round(gu_gbps, 1), "peak": PEAK_GBPS, "unit": "GB/s",
                     "frac": round(gu_gbps / PEAK_GBPS, 4),
                     "traffic": load_traffic("gateup_gemv", wl.name),
                     "algorithmic_bytes": sp0["gateup_bytes_per_launch"],
                     "avg_launch_us": sp0["gateup_avg_launch_us"],
                     "launches_timed": sp0["gateup_launches_timed"]},
        "cpu_baseline": None,
    }
    if dense is not None:
        line["dense_ms_per_token"] = dense["ms_per_token"]
        line["speedup_vs_dense"] = round(dense["ms_per_token"] / mean_sparse, 4)
        line["dense_us_per_layer"] = dense["us_per_layer"]
        line["byte_ratio_sparse_over_dense"] = round(sp0["bytes"] / dense["bytes"], 4)
        line["time_ratio_sparse_over_dense"] = round(sp0["ms_per_token"] / dense["ms_per_token"], 4)
        bts = np.array([r["bytes"] for r in rows], float)
        tms = np.array([r["ms_per_token"] for r in rows], float)
        slope, icpt = np.polyfit(bts, tms, 1)
        pred = slope * bts + icpt
        ss = float(((tms - tms.mean()) ** 2).sum())
        r2 = 1.0 - float(((tms - pred) ** 2).sum() / ss) if ss > 0 else 1.0
        line["time_vs_bytes"] = {"slope_ms_per_GB": round(slope * 1e9, 4),
                                 "intercept_ms": round(icpt, 4), "r2": round(r2, 4),
                                 "bandwidth_of_slope_GBps": round(1.0 / slope / 1e6, 1) if slope > 0 else None}
    return line


def stack_cpu_baseline(args, wl):
    """The oracle on layer 0 of the stack's shape under the first mask, times the layer count (a
    whole stack in float64 does not fit host memory); LM head excluded."""
    import synth
    sh, pos = wl.shape, wl.pos
    sh1 = sh.with_layers(1, vocab=0)
    t0 = time.time()
    layer = synth.layer_weights(sh1, 0)
    m = synth.budget_mask(sh, wl.mask_seeds[0])
    m1 = tuple(a[:1] for a in m)
    prior = synth.kv_prior(sh1, 0, 1, pos, pos + 1)
    x = synth.activations(1, sh.d_model)
    print(f"[bench] CPU oracle layer drawn in {time.time() - t0:.1f}s", file=sys.stderr, flush=True)
    cb = cpu_baseline(sh1, layer, m1, prior, x, pos, args.cpu_seconds)
    cb["per_layer_ms"] = round(cb["value"], 3)
    cb["value"] = round(cb["value"] * sh.n_layers, 3)
    cb["sample"] = (cb["sample"].replace("of the same layer", "of layer 0 of this shape") +
                    f"; times {sh.n_layers} layers, LM head excluded")
    return cb


def bench_stack(args, wl):
    import torch
    from paper_2609_29499_amd import binding as B
    t0 = time.time()
    rows = measure_stack(args, wl.shape, wl.pos, wl.mask_seeds)
    line = stack_line(args, wl, rows)
    # the plain 1 GiB copy: a bandwidth reference, and the calibration of counter runs
    probe = copy_probe_gbps(torch, B)
    line["copy_probe_GBps"] = round(probe, 1)
    line["frac_of_copy_probe"] = round(line["achieved_GBps"] / probe, 4)
    print(f"[bench] {wl.name}: timing done in {time.time() - t0:.1f}s", file=sys.stderr, flush=True)
    if not args.no_cpu:
        line["cpu_baseline"] = stack_cpu_baseline(args, wl)
    if wl.name == "llama3_70b_stack" and not args.no_extras and not args.sparse_only:
        line["extras"] = default_extras(args)
    line["manifest"] = run_manifest()
    print(json.dumps(line), flush=True)


def default_extras(args):
    """The Llama-3-8B-shaped single layer (2048 prior positions) and 32-layer stack (4096) at
    batch 1, sparse vs dense, with the same timing protocol (no CPU baseline, no control)."""
    import copy
    import synth
    ex = {}
    a = copy.copy(args)
    a.no_cpu, a.control = True, False
    t0 = time.time()
    ln = bench_layer(a, synth.WORKLOADS["llama3_8b_layer"])
    ex["llama3_8b_layer"] = {k: ln[k] for k in (
        "value", "unit", "us_per_layer", "dense_ms_per_token", "speedup_vs_dense",
        "byte_ratio_sparse_over_dense", "time_ratio_sparse_over_dense", "achieved_GBps",
        "hbm_frac", "blocks_mean_sd_ms", "kernels_us", "roofline")}
    ex["llama3_8b_layer"]["config"] = ln["config"]
    print(f"[bench] extra 8B layer in {time.time() - t0:.1f}s", file=sys.stderr, flush=True)
    t0 = time.time()
    wl = synth.WORKLOADS["llama3_8b_stack"]
    sl = stack_line(a, wl, measure_stack(a, wl.shape, wl.pos, wl.mask_seeds))
    ex["llama3_8b_stack"] = {k: sl.get(k) for k in (
        "value", "unit", "us_per_layer", "dense_ms_per_token", "speedup_vs_dense",
        "dense_us_per_layer", "achieved_GBps", "hbm_frac", "time_vs_bytes", "roofline")}
    ex["llama3_8b_stack"]["plans"] = [{k: r[k] for k in ("plan", "ms_per_token", "bytes", "GBps",
                                                         "us_per_layer", "active_flop_ratio")}
                                      for r in sl["plans"]]
    ex["llama3_8b_stack"]["config"] = sl["config"]
    print(f"[bench] extra 8B stack in {time.time() - t0:.1f}s", file=sys.stderr, flush=True)
    return ex


KERNEL_SOURCES = {
    "gateup_gemv": ["paper_2609_29499_amd/csrc/gemv_kernels.hip",
                    "paper_2609_29499_amd/csrc/device_common.hpp"],
    "gateup_mfma": ["paper_2609_29499_amd/csrc/mfma_kernels.hip",
                    "paper_2609_29499_amd/csrc/device_common.hpp"],
    "attention": ["paper_2609_29499_amd/csrc/attn_kernels.hip",
                  "paper_2609_29499_amd/csrc/device_common.hpp"],
}


def prefill_flops(sh, counts, T, pos0=0):
    """Algorithmic FLOPs of one prefill of T tokens of one layer: every retained panel weight is
    one multiply-add per token; causal attention is 2 d_h multiply-adds per (query, visible row)
    per retained head (scores and P V)."""
    m_q, m_kv, c = counts
    d, dh = sh.d_model, sh.head_dim
    proj = 2 * T * ((m_q + 2 * m_kv) * dh * d + d * m_q * dh + 3 * d * c)
    visible = sum(pos0 + t + 1 for t in range(T))
    attn = 4 * dh * m_q * visible
    gateup = 2 * T * 2 * c * d
    return {"projections": proj, "attention": attn, "total": proj + attn, "gateup": gateup}


def bench_prefill(args, wl):
    """Prefill of wl.prefill_tokens tokens of one sequence into an empty cache through one layer:
    ms per prefill for the sparse and the dense plan, MFMA throughput on algorithmic FLOPs."""
    import torch
    import synth
    from paper_2609_29499_amd import session as S
    sh, T = wl.shape, wl.prefill_tokens
    t_setup = time.time()
    layer = synth.layer_weights(sh, 0)
    mask = synth.budget_mask(sh, args.mask_seed)
    x = synth.activations(T, sh.d_model, 1)
    desc = S.desc_from_shape(sh, max_batch=1, max_seq=T, max_prefill=T)
    dstore = S.DeviceStore([layer])
    xd = torch.from_numpy(x).cuda()
    out = torch.empty_like(xd)
    results = {}
    for name, m in (("sparse", mask), ("dense", None)):
        probe = S.Plan(desc, dstore, m)
        counts = probe.counts(0)
        del probe
        nb = layer_bytes(sh, *counts, 0)
        copies = max(2, math.ceil(ROTATE_BYTES / nb["weights"]))
        plans = [S.Plan(desc, dstore, m) for _ in range(copies)]
        caches = [S.KVCache(desc, 1, T) for _ in range(copies)]
        for p, c in zip(plans, caches):
            p.prefill(xd, T, c, 0, out)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        st = torch.cuda.Stream()
        st.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(st):
            for p, c in zip(plans, caches):
                p.prefill(xd, T, c, 0, out, stream=S.current_stream())
        torch.cuda.current_stream().wait_stream(st)
        torch.cuda.synchronize()
        with torch.cuda.graph(g):
            for p, c in zip(plans, caches):
                p.prefill(xd, T, c, 0, out, stream=S.current_stream())
        reps = max(1, args.steps // copies)
        for _ in range(max(1, args.warmup // copies)):
            g.replay()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            g.replay()
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / (reps * copies)
        kt = {}
        for i in range(2 * copies):
            for kname, kms in plans[i % copies].prefill_timed(xd, T, caches[i % copies], 0, out):
                kt.setdefault(kname, []).append(kms)
        kt = {k: float(np.mean(v)) for k, v in kt.items()}
        fl = prefill_flops(sh, counts, T)
        results[name] = {"counts": counts, "ms": ms, "kernels": kt, "flops": fl, "copies": copies,
                         "steps": reps * copies}
        print(f"[bench] prefill {name}: {ms:.3f} ms, {fl['total'] / (ms * 1e-3) / 1e12:.1f} TFLOP/s, "
              f"kernels(us)=" + " ".join(f"{k}={v*1e3:.1f}" for k, v in kt.items()),
              file=sys.stderr, flush=True)
        del g, plans, caches
        torch.cuda.empty_cache()
    sp, dn = results["sparse"], results["dense"]
    gu_ms = sp["kernels"]["gateup_gemm"]
    gu_tf = sp["flops"]["gateup"] / (gu_ms * 1e-3) / 1e12
    line = {
        "metric": METRIC, "value": round(sp["ms"], 5), "unit": "ms/prefill", "n_gpus": 1,
        "steps": sp["steps"], "warmup": args.warmup, "ms_per_step": round(sp["ms"], 5),
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "int8w-int8x3-f32",
        "data": "synthetic",
        "config": {"workload": wl.name, "d_model": sh.d_model, "n_q_heads": sh.n_q_heads,
                   "n_kv_heads": sh.n_kv_heads, "head_dim": sh.head_dim, "d_ffn": sh.d_ffn,
                   "layers": 1, "tokens": T, "pos0": 0, "mask_seed": args.mask_seed,
                   "retained": {"q_heads": sp["counts"][0], "kv_groups": sp["counts"][1],
                                "ffn_channels": sp["counts"][2]}},
        "tokens_per_s": round(T / (sp["ms"] * 1e-3), 1),
        "algorithmic_TFLOPs": round(sp["flops"]["total"] / (sp["ms"] * 1e-3) / 1e12, 2),
        "dense_ms_per_prefill": round(dn["ms"], 5),
        "speedup_vs_dense": round(dn["ms"] / sp["ms"], 4),
        "flop_ratio_sparse_over_dense": round(sp["flops"]["total"] / dn["flops"]["total"], 4),
        "kernels_us": {k: {n: round(v * 1e3, 2) for n, v in r["kernels"].items()} for k, r in results.items()},
        "roofline": {"bound": "mfma", "kernel": "gateup_gemm", "achieved": round(gu_tf, 1),
                     "peak": 2500.0, "unit": "TFLOP/s", "frac": round(gu_tf / 2500.0, 4),
                     "issued_frac": round(3 * gu_tf / 5000.0, 4), "traffic": None,
                     "algorithmic_flops": sp["flops"]["gateup"], "avg_launch_us": round(gu_ms * 1e3, 2),
                     "note": "activations as three INT8 digits: three INT8 passes (issued_frac against 5000 TOP/s)"},
        "paper_context": "prefill 1814 -> 1326 ms (2048 tokens, 80 layers, dense vs sparse, A100)",
    }
    print(f"[bench] setup+timing {time.time() - t_setup:.1f}s", file=sys.stderr, flush=True)
    if not args.no_cpu:
        line["cpu_baseline"] = cpu_prefill_baseline(sh, layer, mask, x, args.cpu_seconds)
    else:
        line["cpu_baseline"] = None
    print(json.dumps(line), flush=True)


def cpu_prefill_baseline(sh, store_layer, mask, x, budget_s):
    import threadpoolctl
    from oracle import reference as ref
    closed = ref.close_mask(*mask, sh.group_size)
    W = ref.masked_layer(store_layer, closed[0][0], closed[1][0], closed[2][0], sh.head_dim)
    T = x.shape[0]
    times = []
    t_start = time.perf_counter()
    while time.perf_counter() - t_start < budget_s or len(times) < 1:
        K = np.zeros((sh.n_kv_heads, T, sh.head_dim))
        V = np.zeros_like(K)
        t0 = time.perf_counter()
        ref.prefill_layer(W, x, K, V, 0, sh)
        times.append(time.perf_counter() - t0)
    info = threadpoolctl.threadpool_info()
    threads = max([i.get("num_threads", 1) for i in info] or [1])
    return {"value": float(np.median(times) * 1e3), "unit": "ms/prefill", "cores": int(threads),
            "kind": "oracle",
            "sample": f"{len(times)} oracle prefills of the same layer and {T} tokens (float64 numpy, "
                      f"zero-masked dequantised weights resident), median",
            "host_cpus": len(os.sched_getaffinity(0))}


def bench_request(args, wl):
    """The paper's timed request shape under one plan: embed a seeded prompt, prefill it, then
    wl.n_new greedy decode steps with device-side ids (tasp_generate), for the dense plan and the
    seed-1 mask. Reports prefill ms, decode ms per token and the whole request."""
    import torch
    import synth
    from paper_2609_29499_amd import session as S
    sh, T, n_new = wl.shape, wl.prefill_tokens, wl.n_new
    gen = torch.Generator(device="cuda")
    gen.manual_seed(0)
    t0 = time.time()
    layers = [device_layer(torch, sh, gen) for _ in range(sh.n_layers)]
    fnorm = (1.0 + 0.1 * torch.randn(sh.d_model, generator=gen, device="cuda")).to(torch.bfloat16).view(torch.int16)
    lm = (0.02 * torch.randn(sh.vocab, sh.d_model, generator=gen, device="cuda")).to(torch.bfloat16).view(torch.int16)
    e = torch.randn(sh.vocab, sh.d_model, generator=gen, device="cuda")
    e_scale = (e.abs().amax(dim=1) / 127.0).clamp_min(1e-30)
    embed = torch.round(e / e_scale[:, None]).clamp_(-127, 127).to(torch.int8)
    del e
    store = S.DeviceStore(layers, fnorm, lm)
    desc = S.desc_from_shape(sh, max_batch=1, max_seq=T + n_new, max_prefill=T)
    prompt = torch.from_numpy(synth.prompt_ids(T, sh.vocab)).cuda()
    torch.cuda.synchronize()
    print(f"[bench] {wl.name}: store drawn in {time.time() - t0:.1f}s", file=sys.stderr, flush=True)
    rows = []
    for name, m in (("dense", None), ("mask1", synth.budget_mask(sh, args.mask_seed))):
        plan = S.Plan(desc, store, m)
        cache = S.KVCache(desc, 1, T + n_new)
        scratch = (torch.empty((T, sh.d_model), device="cuda"), torch.empty((T, sh.vocab), device="cuda"))
        plan.generate(embed, e_scale, prompt, n_new, cache, scratch=scratch)      # warm-up
        torch.cuda.synchronize()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        req, pf = [], []
        for _ in range(max(1, args.steps)):
            ev[0].record()
            ids = plan.generate(embed, e_scale, prompt, n_new, cache, scratch=scratch)
            ev[1].record()
            torch.cuda.synchronize()
            req.append(ev[0].elapsed_time(ev[1]))
            # the prefill alone as the request runs it (the same embedded prompt; the last
            # token's logits only)
            ev[2].record()
            plan.prefill_last(scratch[0], T, cache, 0, scratch[1][T - 1])
            ev[3].record()
            torch.cuda.synchronize()
            pf.append(ev[2].elapsed_time(ev[3]))
            print(f"[bench] {name}: request {len(req)}: {req[-1]:.1f} ms", file=sys.stderr, flush=True)
        req_ms, pf_ms = float(np.median(req)), float(np.median(pf))
        dec = (req_ms - pf_ms) / n_new
        rows.append({"plan": name, "request_ms": round(req_ms, 3), "prefill_ms": round(pf_ms, 3),
                     "decode_ms_per_token": round(dec, 4), "first_ids": ids[:4].cpu().tolist(),
                     "active_flop_ratio": round(plan.ledger()["active_flop_ratio"], 4)})
        print(f"[bench] {name}: request {req_ms:.1f} ms, prefill {pf_ms:.2f} ms, decode {dec:.3f} ms/token",
              file=sys.stderr, flush=True)
        del plan, cache, scratch
        torch.cuda.empty_cache()
    dn, sp = rows
    line = {
        "metric": METRIC, "value": sp["decode_ms_per_token"], "unit": "ms/token", "n_gpus": 1,
        "steps": max(1, args.steps), "warmup": 1, "ms_per_step": sp["decode_ms_per_token"],
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "int8w-f32",
        "data": "synthetic",
        "config": {"workload": wl.name, "d_model": sh.d_model, "layers": sh.n_layers,
                   "vocab": sh.vocab, "prompt_tokens": T, "decode_steps": n_new, "batch": 1},
        "dense_ms_per_token": dn["decode_ms_per_token"],
        "speedup_vs_dense": round(dn["decode_ms_per_token"] / sp["decode_ms_per_token"], 4),
        "prefill_ms": {"dense": dn["prefill_ms"], "sparse": sp["prefill_ms"]},
        "request_ms": {"dense": dn["request_ms"], "sparse": sp["request_ms"]},
        "plans": rows, "roofline": None, "cpu_baseline": None,
        "paper_context": "Llama-3-70B on one A100: decode 45.2 -> 31.3 ms/token, prefill (2048 tokens) "
                         "1814 -> 1326 ms, dense vs compiled sparse",
    }
    print(json.dumps(line), flush=True)


def bench_mask(args, wl):
    """Greedy dependency-closed mask construction from seeded scores: ms per build on the GPU
    (each call synchronises), checked against the oracle, with the oracle timed on the host."""
    import torch
    from paper_2609_29499_amd import session as S
    sh, granule = wl.shape, wl.granule
    rng = np.random.default_rng(args.mask_seed)
    hs = rng.uniform(0, 1, (sh.n_layers, sh.n_q_heads)).astype(np.float32)
    cs = rng.uniform(0, 1, (sh.n_layers, sh.d_ffn // granule)).astype(np.float32)
    desc = S.desc_from_shape(sh)
    hd, cd = torch.from_numpy(hs).cuda(), torch.from_numpy(cs).cuda()
    for _ in range(max(1, args.warmup)):
        q, kv, f, spent = S.build_mask(desc, hd, cd, granule, 0.57)
    torch.cuda.synchronize()
    reps = max(1, args.steps)
    t0 = time.perf_counter()
    for _ in range(reps):
        q, kv, f, spent = S.build_mask(desc, hd, cd, granule, 0.57)
    ms = (time.perf_counter() - t0) / reps * 1e3
    cpu = None
    if not args.no_cpu:
        # CPU baseline: the oracle's construction of the same candidate set, timed once; its
        # selection is reported next to the GPU's
        from oracle import greedy as G
        t1 = time.perf_counter()
        wq, wkv, wf, wspent, _ = G.greedy_mask(sh, hs, cs, granule, 0.57)
        cpu_ms = (time.perf_counter() - t1) * 1e3
        same = (spent == wspent and np.array_equal(q.cpu().numpy(), wq)
                and np.array_equal(kv.cpu().numpy(), wkv) and np.array_equal(f.cpu().numpy(), wf))
        cpu = {"value": round(cpu_ms, 3), "unit": "ms/mask", "cores": 1, "kind": "oracle",
               "sample": "one oracle construction of the same candidate set (Python loop)",
               "same_selection_as_gpu": bool(same)}
    n_cand = sh.n_layers * (sh.n_q_heads + sh.d_ffn // granule)
    line = {
        "metric": "ms per greedy dependency-closed mask construction", "value": round(ms, 4),
        "unit": "ms/mask", "n_gpus": 1, "steps": reps, "warmup": args.warmup, "ms_per_step": round(ms, 4),
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "f64-keys/int64-costs",
        "data": "synthetic",
        "config": {"workload": wl.name, "layers": sh.n_layers, "candidates": n_cand,
                   "granule": granule, "target": 0.57},
        "active_flop_ratio": round(spent / dense_layer_flops(sh), 6),
        "roofline": None,
        "cpu_baseline": cpu,
    }
    print(json.dumps(line), flush=True)


def shared_ledger(S, B, sh, seeds):
    """Device bytes at the paper's request shape (2,048-token prefill + 256 decode steps, batch
    1) from the library's workspace queries (no allocation): the groupwise store, 1 .. len(seeds)
    shared-store plans (fixed metadata each) over one scratch arena and the KV cache, against
    materialised plans (each holds its own panels and scratch; their store can be freed)."""
    import synth
    d, dh, F = sh.d_model, sh.head_dim, sh.d_ffn
    per_layer = ((sh.n_q_heads + 2 * sh.n_kv_heads) * dh * d + d * sh.n_q_heads * dh + 3 * F * d)
    weights = sh.n_layers * per_layer
    scales = weights // 128 * 2
    gains = sh.n_layers * 2 * d * 2 + (d * 2 + sh.vocab * d * 2 if sh.vocab else 0)
    S_ = 2048 + 256
    desc = S.desc_from_shape(sh, max_batch=1, max_seq=S_, max_prefill=2048)
    plan_b, arena_b = B.tasp_shared_plan_workspace_bytes(desc)
    kv = 2 * sh.n_layers * sh.n_kv_heads * S_ * dh * 2
    mats = []
    for sd in seeds:
        mptr, keep = S.mask_struct(synth.budget_mask(sh, sd))
        mats.append(B.tasp_plan_workspace_bytes(desc, mptr))
    rows = []
    for n in (1, 3, len(seeds)):
        rows.append({"masks": n,
                     "shared_GB": round((weights + scales + gains + n * plan_b + arena_b + kv) / 1e9, 3),
                     "shared_metadata_GB": round(n * plan_b / 1e9, 4),
                     "materialised_GB": round((sum(mats[:n]) + kv) / 1e9, 3)})
    return {"store_weight_GB": round(weights / 1e9, 3), "store_scale_GB": round(scales / 1e9, 3),
            "gains_and_lm_head_GB": round(gains / 1e9, 3), "kv_cache_GB": round(kv / 1e9, 3),
            "plan_MB": round(plan_b / 1e6, 2), "shared_scratch_arena_MB": round(arena_b / 1e6, 1),
            "by_masks": rows,
            "note": "max_seq 2304, max_prefill 2048, batch 1; every shared plan uses one scratch arena"}


def bench_shared(args, wl):
    """Batch-1 decode of one layer from shared-store plans (groupwise INT8, BF16 scales per 128
    inputs; plans are maps into the store) against the materialised per-row plan of the same
    mask, with every timed step reading its weights from HBM (rotation over store copies), the
    shared gate/up kernel's roofline, and the memory ledger at the 8B and 70B shapes."""
    import torch
    import synth
    from paper_2609_29499_amd import binding as B
    from paper_2609_29499_amd import session as S
    sh, pos = wl.shape, wl.pos
    t0 = time.time()
    layer_g = synth.layer_weights(sh, 0, quant="group")
    mask = synth.budget_mask(sh, args.mask_seed)
    prior = synth.kv_prior(sh, 0, 1, pos, pos + 1)
    x = synth.activations(1, sh.d_model)
    desc = S.desc_from_shape(sh, max_batch=1, max_seq=pos + 1)
    first = S.GroupStore([layer_g])
    store_bytes = first.nbytes()
    copies = max(2, math.ceil(ROTATE_BYTES / store_bytes))
    stores = [first]
    for _ in range(copies - 1):
        stores.append(S.GroupStore([{k: v for k, v in layer_g.items()}]))
    torch.cuda.synchronize()
    print(f"[bench] {wl.name}: {copies} store copies of {store_bytes / 1e6:.1f} MB in "
          f"{time.time() - t0:.1f}s", file=sys.stderr, flush=True)
    results = {}
    for name, m in (("shared_sparse", mask), ("shared_dense", None)):
        rot = Rotation(S, torch, sh, desc, None, m, prior, x, pos, copies,
                       make_plan=lambda i, m=m: S.Plan.shared(desc, stores[i], m))
        rot.run_steps(args.warmup)
        ms = rot.time_steps(args.steps)
        kt = rot.kernel_times(args.timed_launches)
        st_ms = rot.stage_ms(STAGE_KIND["gateup_gemv"]) if name == "shared_sparse" else None
        counts = rot.plans[0].counts(0)
        results[name] = {"ms": ms, "kernels": kt, "stage_ms": st_ms, "counts": counts,
                         "ledger": rot.plans[0].ledger()}
        print(f"[bench] {name}: {ms * 1e3:.2f} us/step kernels(us)=" +
              " ".join(f"{k}={v * 1e3:.2f}" for k, v in kt.items()), file=sys.stderr, flush=True)
        del rot
        torch.cuda.empty_cache()
    del stores, first
    torch.cuda.empty_cache()
    # the materialised per-row plan of the same mask (the default benchmark's sparse plan)
    layer_r = synth.layer_weights(sh, 0)
    dstore = S.DeviceStore([layer_r])
    probe = S.Plan(desc, dstore, mask)
    nb = layer_bytes(sh, *probe.counts(0), pos, 1)
    mat_ws = probe.ws_bytes
    del probe
    mcopies = max(2, math.ceil(ROTATE_BYTES / nb["total"]))
    rot = Rotation(S, torch, sh, desc, dstore, mask, prior, x, pos, mcopies)
    rot.run_steps(args.warmup)
    mat_ms = rot.time_steps(args.steps)
    del rot
    torch.cuda.empty_cache()
    print(f"[bench] materialised per-row: {mat_ms * 1e3:.2f} us/step", file=sys.stderr, flush=True)
    sp = results["shared_sparse"]
    c = sp["counts"][2]
    d = sh.d_model
    gu_bytes = 2 * c * d + 2 * c * (d // 128) * 2 + d * 4 + c * 4
    gu_gbps = gu_bytes / (sp["stage_ms"] * 1e-3) / 1e9
    line = {
        "metric": METRIC, "value": round(sp["ms"], 6), "unit": "ms/token", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(sp["ms"], 6),
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "int8w-g128-f32",
        "data": "synthetic",
        "config": {"workload": wl.name, "d_model": d, "layers": 1, "batch": 1, "pos": pos,
                   "mask_seed": args.mask_seed, "scales": "BF16 per 128 inputs",
                   "retained": {"q_heads": sp["counts"][0], "kv_groups": sp["counts"][1],
                                "ffn_channels": c}},
        "us_per_layer": {"shared_sparse": round(sp["ms"] * 1e3, 3),
                         "shared_dense": round(results["shared_dense"]["ms"] * 1e3, 3),
                         "materialised_per_row_sparse": round(mat_ms * 1e3, 3)},
        "speedup_vs_shared_dense": round(results["shared_dense"]["ms"] / sp["ms"], 4),
        "kernels_us": {k: {n: round(v * 1e3, 3) for n, v in r["kernels"].items()}
                       for k, r in results.items() if "kernels" in r},
        "roofline": {"bound": "hbm", "kernel": "shared_gateup_gemv", "achieved": round(gu_gbps, 1),
                     "peak": PEAK_GBPS, "unit": "GB/s", "frac": round(gu_gbps / PEAK_GBPS, 4),
                     "traffic": None, "algorithmic_bytes": gu_bytes,
                     "avg_launch_us": round(sp["stage_ms"] * 1e3, 3)},
        "memory": {"layer_store_MB": round(store_bytes / 1e6, 1),
                   "shared_plan_workspace_MB": round(sum(B.tasp_shared_plan_workspace_bytes(desc)) / 1e6, 3),
                   "materialised_plan_workspace_MB": round(mat_ws / 1e6, 1),
                   "llama3_8b": shared_ledger(S, B, synth.LLAMA3_8B, (1, 2, 3, 4, 5)),
                   "llama3_70b": shared_ledger(S, B, synth.LLAMA3_70B, (1, 2, 3, 4, 5))},
        "rotation_copies": {"shared": copies, "materialised": mcopies},
        "paper_context": "one packed store for five 70B masks: 76.9 / 77.1 / 77.3 GB peak for 1 / 3 / 5 "
                         "masks, plan metadata 0.14 / 0.34 / 0.54 GB (A100 runtime)",
    }
    if not args.no_cpu:
        print("[bench] timing the CPU oracle", file=sys.stderr, flush=True)
        line["cpu_baseline"] = cpu_baseline(sh, layer_g, mask, prior, x, pos, args.cpu_seconds)
    else:
        line["cpu_baseline"] = None
    print(json.dumps(line), flush=True)


ROUTER_TAUS = (0.50, 0.70, 0.85, 0.95)
PAPER_USAGE_085 = 0.76       # sparse-path share at tau = 0.85 in the paper's threshold sweep


def bench_router(args, wl):
    """Routing of user turns (tasp_route): per-turn latency on a 2048-token-sized prompt with the
    decision read back by the host, batched throughput over a mix of the five task families,
    sparse-path usage u(tau) of that mix, and the mixture-implied decode latency
    u L_sparse + (1 - u) L_dense with both path latencies measured on the 8B stack in this run.
    The router weights are random (seeded): u(tau) shows the mechanics, not a trained router."""
    import torch
    from paper_2609_29499_amd import session as S
    from synth import text as T
    w = T.router_weights()
    router = S.Router(w, temperature=1.0, tau=0.85)
    # one turn: a 2048-token-sized prompt (about 8 KiB of text)
    turn = T.prompt(31, 0, family=0, n_sent=130)
    tb = torch.from_numpy(np.frombuffer(turn, np.uint8).copy()).cuda()
    lp = torch.tensor([-2.0], device="cuda")
    host = torch.empty(1, dtype=torch.int32).pin_memory()
    reps = max(1, args.steps)

    def one_turn():
        _, _, c = router.route(tb, None, lp, features=False)
        host.copy_(c)                       # the host needs the decision to pick the plan
        return int(host[0])

    for _ in range(max(1, args.warmup)):
        one_turn()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        one_turn()
    turn_ms = (time.perf_counter() - t0) / reps * 1e3
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    ev[0].record()
    for _ in range(reps):
        router.route(tb, None, lp, features=False)
    ev[1].record()
    torch.cuda.synchronize()
    dev_ms = ev[0].elapsed_time(ev[1]) / reps
    print(f"[bench] router turn {turn_ms:.4f} ms (device {dev_ms:.4f} ms, {len(turn)} bytes)",
          file=sys.stderr, flush=True)
    # a batch of turns from the five families
    texts = T.prompts(512, seed=32)
    buf, offs = T.pack(texts)
    btb, bto = torch.from_numpy(buf).cuda(), torch.from_numpy(offs).cuda()
    blp = torch.from_numpy(T.proxy_logprobs(len(texts), seed=33)).cuda()
    for _ in range(3):
        _, probs, _ = router.route(btb, bto, blp, features=False)
    torch.cuda.synchronize()
    ev[0].record()
    for _ in range(max(1, reps // 10)):
        _, probs, _ = router.route(btb, bto, blp, features=False)
    ev[1].record()
    torch.cuda.synchronize()
    batch_ms = ev[0].elapsed_time(ev[1]) / max(1, reps // 10)
    # No labelled prompts exist here to fit the temperature on, so it is set so that the mix uses
    # the sparse path on the paper's share of turns at tau = 0.85 (76%): softmax(z / t) is
    # softmax(log p / t) for the probabilities p at temperature 1, so the fit needs no logits.
    logp = np.log(np.maximum(probs.double().cpu().numpy(), 1e-300))

    def usage_at(temp, tau):
        u = logp / temp
        u = np.exp(u - u.max(axis=1, keepdims=True))
        return float(((u / u.sum(axis=1, keepdims=True)).max(axis=1) >= tau).mean())

    lo, hi = 1e-4, 1.0
    for _ in range(60):
        mid = np.sqrt(lo * hi)
        lo, hi = (mid, hi) if usage_at(mid, 0.85) > PAPER_USAGE_085 else (lo, mid)
    temp = float(np.sqrt(lo * hi))
    fitted = S.Router(w, temperature=temp, tau=0.85)
    _, probs, choice = fitted.route(btb, bto, blp, features=False)
    pmax = probs.max(dim=1).values.cpu().numpy()
    used = {t: float((pmax >= np.float32(t)).mean()) for t in ROUTER_TAUS}
    # the kernel's own decisions at tau = 0.85 agree with its probabilities
    assert used[0.85] == float((choice.cpu().numpy() >= 0).mean())
    usage = {f"{t:.2f}": round(u, 4) for t, u in used.items()}
    # the two path latencies the mixture is formed from
    rows = measure_stack(args, wl.shape, wl.pos, wl.mask_seeds)
    l_sparse = rows[0]["ms_per_token"]
    l_dense = next(r["ms_per_token"] for r in rows if r["plan"] == "dense")
    # mixture-implied latency at sparse-path usage u: u L_sparse + (1 - u) L_dense
    mixture = {t: round(u * l_sparse + (1.0 - u) * l_dense, 5) for t, u in usage.items()}
    # CPU baseline: the oracle on the host, features + MLP of the same turn, for about cpu_seconds
    from oracle import router as R
    t1 = time.perf_counter()
    n_cpu = 0
    while time.perf_counter() - t1 < min(args.cpu_seconds, 10.0) or n_cpu == 0:
        R.route(turn, -2.0, w, 1.0, 0.85)
        n_cpu += 1
    cpu_ms = (time.perf_counter() - t1) / n_cpu * 1e3
    line = {
        "metric": "router ms per user turn (features + MLP + decision on the host)",
        "value": round(turn_ms, 5), "unit": "ms/turn", "n_gpus": 1, "steps": reps,
        "warmup": args.warmup, "ms_per_step": round(turn_ms, 5), "higher_is_better": False,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": wl.name, "n_bins": 2048, "proj_dim": 256, "hidden": [512, 256],
                   "n_tasks": 5, "tau": 0.85, "turn_bytes": len(turn), "batch_prompts": len(texts),
                   "stack": {"d_model": wl.shape.d_model, "layers": wl.shape.n_layers,
                             "pos": wl.pos, "mask": wl.mask_seeds[0]}},
        "device_ms_per_turn": round(dev_ms, 5),
        "batch_ms": round(batch_ms, 4),
        "batch_turns_per_s": round(len(texts) / (batch_ms * 1e-3), 1),
        "temperature": round(temp, 6),
        "temperature_note": "random router: temperature set so that the mix's sparse-path share "
                            "at tau 0.85 matches the paper's 76% (no labels to fit it on)",
        "sparse_usage": usage,
        "decode_ms_per_token": {"sparse": l_sparse, "dense": l_dense},
        "mixture_ms_per_token": mixture,
        "roofline": None,
        "roofline_note": "five small launches per turn (about 1 MFLOP and 3.2 MB of float32 "
                         "weights): bound by launch and dependency latency, not by a unit's peak",
        "cpu_baseline": {"value": round(cpu_ms, 4), "unit": "ms/turn", "cores": 1,
                         "kind": "oracle", "sample": f"{n_cpu} routings of the same "
                         f"{len(turn)}-byte turn (Python text scan + float64 MLP)"},
        "paper_context": "router + features 0.16 +- 0.02 ms per turn; mixture-implied decode "
                         "32.6 / 34.6 / 38.0 ms/token at tau 0.70 / 0.85 / 0.95 (Llama-3-70B, A100)",
    }
    print(json.dumps(line), flush=True)


def mask_as_zero_control(args, S, B, torch, sh, desc, dstore, layer, mask, prior, x, pos, batch):
    """The paper's mask-as-zero control: the same mask applied as zeros in the dense store, run as
    a dense plan (dense launch shapes, same result as the compiled plan). The keep bits come from
    the compiled plan's own index lists."""
    import synth

    probe = S.Plan(desc, dstore, mask)
    keep = [np.zeros(n, bool) for n in (sh.n_q_heads, sh.n_kv_heads, sh.d_ffn)]
    for k, which in zip(keep, (B.IDX_Q, B.IDX_KV, B.IDX_FFN)):
        k[probe.indices(0, which)] = True
    del probe
    zstore = S.DeviceStore([synth.zero_dropped(layer, sh, *keep)])
    nb = layer_bytes(sh, sh.n_q_heads, sh.n_kv_heads, sh.d_ffn, pos, batch)
    copies = max(2, math.ceil(ROTATE_BYTES / nb["total"]))
    rot = Rotation(S, torch, sh, desc, zstore, None, prior, x, pos, copies)
    rot.run_steps(args.warmup)
    torch.cuda.synchronize()
    ms = rot.time_steps(args.steps)
    print(f"[bench] mask as zero (dense plan, zeroed store): {ms*1e3:.2f} us/step",
          file=sys.stderr, flush=True)
    del rot, zstore
    torch.cuda.empty_cache()
    return {"ms": ms, "copies": copies}


def load_traffic(kernel, workload):
    """HBM bytes per launch of a kernel from the committed counter summary of this workload, if
    the counters were taken on the current kernel source; else None."""
    p = os.path.join(ROOT, "profiles", f"{kernel}_{workload}_traffic.json")
    if not os.path.exists(p) or kernel not in KERNEL_SOURCES:
        return None
    with open(p) as f:
        t = json.load(f)
    if t.get("kernel_source_hash") != source_hash(KERNEL_SOURCES[kernel]):
        return None
    return t.get("bytes_per_launch")


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU only; --gpus must be 1"}))
        sys.exit(2)
    import torch

    import synth
    from paper_2609_29499_amd import binding as B
    from paper_2609_29499_amd import session as S

    if not torch.cuda.is_available():
        print(json.dumps({"error": "no GPU visible"}))
        sys.exit(1)
    B.load()
    wl = synth.WORKLOADS[args.workload]
    sh, pos = wl.shape, wl.pos
    if wl.kind == "mask":
        bench_mask(args, wl)
        return
    if wl.kind == "request":
        bench_request(args, wl)
        return
    if wl.kind == "router":
        bench_router(args, wl)
        return
    if wl.kind == "shared":
        (bench_shared_stack if sh.n_layers > 1 else bench_shared)(args, wl)
        return
    if sh.n_layers > 1 and wl.batch == 1 and wl.prefill_tokens == 0:
        bench_stack(args, wl)
        return
    if wl.prefill_tokens:
        bench_prefill(args, wl)
        return
    if sh.n_layers != 1 or wl.prefill_tokens:
        print(json.dumps({"error": f"workload {args.workload} is not a single-layer decode"}))
        sys.exit(2)
    line = bench_layer(args, wl)
    if line is not None:
        line["manifest"] = run_manifest()
        print(json.dumps(line), flush=True)


def bench_layer(args, wl):
    """One decoder layer (batch 1 or 8) over rotating plan copies: the sparse plan of the seed
    mask and the dense plan. Returns the JSON line (None for --sparse-only counter runs, which
    print their own summary)."""
    import torch

    import synth
    from paper_2609_29499_amd import binding as B
    from paper_2609_29499_amd import session as S
    sh, pos = wl.shape, wl.pos
    batch = wl.batch
    t_setup = time.time()
    print(f"[bench] generating {wl.name}", file=sys.stderr, flush=True)
    layer = synth.layer_weights(sh, 0)
    mask = synth.budget_mask(sh, args.mask_seed)
    prior = synth.kv_prior(sh, 0, batch, pos, pos + 1)
    x = synth.activations(batch, sh.d_model)
    desc = S.desc_from_shape(sh, max_batch=batch, max_seq=pos + 1)
    dstore = S.DeviceStore([layer])
    results = {}
    plans = (("sparse", mask),) if args.sparse_only else (("sparse", mask), ("dense", None))
    # the kernel that moves the most bytes: the gate/up panels at batch 1, the KV cache at batch 8
    probe_counts = S.Plan(desc, dstore, mask).counts(0)
    nb0 = layer_bytes(sh, *probe_counts, pos, batch)
    dominant = "attention" if nb0["attention"] > nb0["gateup"] else "gateup_gemv"
    for name, m in plans:
        probe = S.Plan(desc, dstore, m)
        counts = probe.counts(0)
        ledger = probe.ledger()
        del probe
        nb = layer_bytes(sh, *counts, pos, batch)
        copies = max(2, math.ceil(ROTATE_BYTES / nb["total"]))
        print(f"[bench] {name}: counts={counts} bytes={nb['total']/1e6:.1f} MB copies={copies}",
              file=sys.stderr, flush=True)
        rot = Rotation(S, torch, sh, desc, dstore, m, prior, x, pos, copies)
        rot.run_steps(args.warmup)
        torch.cuda.synchronize()
        ms = rot.time_steps(args.steps)
        blocks = [rot.time_steps(200) for _ in range(args.blocks)]
        eager = rot.time_eager(max(200, args.steps // 5))
        ktimes = rot.kernel_times(args.timed_launches)
        stage_ms = rot.stage_ms(STAGE_KIND[dominant])
        results[name] = {"counts": counts, "ledger": ledger, "bytes": nb, "ms": ms,
                         "blocks": blocks, "eager": eager, "kernels": ktimes, "copies": copies,
                         "stage_ms": stage_ms}
        print(f"[bench] {name}: {ms*1e3:.2f} us/step  kernels(us)=" +
              " ".join(f"{k}={v*1e3:.2f}" for k, v in ktimes.items()), file=sys.stderr, flush=True)
        del rot
        torch.cuda.empty_cache()
    if not args.sparse_only and getattr(args, "control", True):
        results["mask_as_zero"] = mask_as_zero_control(args, S, B, torch, sh, desc, dstore, layer,
                                                       mask, prior, x, pos, batch)
    probe = copy_probe_gbps(torch, B)
    if args.sparse_only:
        print(json.dumps({"sparse_ms_per_step": results["sparse"]["ms"],
                          "kernels_us": {k: v * 1e3 for k, v in results["sparse"]["kernels"].items()},
                          "copy_probe_GBps": probe}), flush=True)
        return None
    sp, dn = results["sparse"], results["dense"]
    sp_block = float(np.mean(sp["blocks"])) if sp["blocks"] else sp["ms"]
    dn_block = float(np.mean(dn["blocks"])) if dn["blocks"] else dn["ms"]
    st_ms = sp["stage_ms"]
    st_bytes = sp["bytes"]["attention" if dominant == "attention" else "gateup"]
    st_gbps = st_bytes / (st_ms * 1e-3) / 1e9
    traffic = load_traffic("gateup_mfma" if dominant == "gateup_gemv" and batch > 1 else dominant,
                           wl.name)
    gbps = sp["bytes"]["total"] / (sp_block * 1e-3) / 1e9
    line = {
        "metric": METRIC, "value": round(sp_block, 6), "unit": "ms/token", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(sp["ms"], 6),
        "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "int8w-f32",
        "data": "synthetic",
        "config": {"workload": wl.name, "d_model": sh.d_model, "n_q_heads": sh.n_q_heads,
                   "n_kv_heads": sh.n_kv_heads, "head_dim": sh.head_dim, "d_ffn": sh.d_ffn,
                   "layers": 1, "batch": batch, "pos": pos, "mask_seed": args.mask_seed,
                   "active_flop_ratio": round(sp["ledger"]["active_flop_ratio"], 4),
                   "retained": {"q_heads": sp["counts"][0], "kv_groups": sp["counts"][1],
                                "ffn_channels": sp["counts"][2]}},
        "value_protocol": f"mean of {len(sp['blocks'])} blocks x 200 graph-replayed steps",
        "us_per_layer": round(sp_block * 1e3, 3),
        "dense_ms_per_token": round(dn_block, 6),
        "speedup_vs_dense": round(dn_block / sp_block, 4),
        "byte_ratio_sparse_over_dense": round(sp["bytes"]["total"] / dn["bytes"]["total"], 4),
        "time_ratio_sparse_over_dense": round(sp_block / dn_block, 4),
        "achieved_GBps": round(gbps, 1), "hbm_frac": round(gbps / PEAK_GBPS, 4),
        "copy_probe_GBps": round(probe, 1), "frac_of_copy_probe": round(gbps / probe, 4),
        "dense_achieved_GBps": round(dn["bytes"]["total"] / (dn_block * 1e-3) / 1e9, 1),
        "step_bytes": {"sparse": sp["bytes"]["total"], "dense": dn["bytes"]["total"]},
        "blocks_ms": {"sparse": [round(b, 6) for b in sp["blocks"]],
                      "dense": [round(b, 6) for b in dn["blocks"]]},
        "blocks_mean_sd_ms": {k: [round(float(np.mean(r["blocks"])), 6),
                                  round(float(np.std(r["blocks"], ddof=1)), 6)]
                              for k, r in (("sparse", sp), ("dense", dn)) if len(r["blocks"]) > 1},
        "plain_launch_ms_per_token": {"sparse": round(sp["eager"], 6),
                                      "dense": round(dn["eager"], 6)},
        "kernels_us": {k: {n: round(v * 1e3, 3) for n, v in r["kernels"].items()}
                       for k, r in results.items() if "kernels" in r},
        "roofline": {"bound": "hbm", "kernel": dominant, "achieved": round(st_gbps, 1),
                     "peak": PEAK_GBPS, "unit": "GB/s", "frac": round(st_gbps / PEAK_GBPS, 4),
                     "traffic": traffic, "algorithmic_bytes": st_bytes,
                     "avg_launch_us": round(st_ms * 1e3, 3)},
        "paper_context": "45.2 -> 31.3 ms/token dense vs compiled sparse, Llama-3-70B, INT8/BF16, one A100 80GB",
        "rotation_copies": {"sparse": sp["copies"], "dense": dn["copies"]},
    }
    if "mask_as_zero" in results:
        line["mask_as_zero"] = {"ms_per_token": round(results["mask_as_zero"]["ms"], 6),
                                "speedup_vs_dense": round(dn["ms"] / results["mask_as_zero"]["ms"], 4),
                                "paper_context": "mask-as-zero 1.03x vs compiled 1.44x over dense "
                                                 "(Llama-3-70B, one A100)"}
    print(f"[bench] setup+timing {time.time()-t_setup:.1f}s", file=sys.stderr, flush=True)
    if not args.no_cpu:
        print("[bench] timing the CPU oracle", file=sys.stderr, flush=True)
        line["cpu_baseline"] = cpu_baseline(sh, layer, mask, prior, x, pos, args.cpu_seconds)
    else:
        line["cpu_baseline"] = None
    return line


if __name__ == "__main__":
    main()
