"""Timed cases of the eviction + ragged-decode path, through the calls of paper_2506_15724_amd.binding.

A case is a model shape (layers, batch, heads, head_dim, context, window, budget), the options of the reduced cache
and what a pass does with it:

  op "evict"    madakv_evict over the prompt, `layers_per_call` layers at a time, then `steps` decode steps, one
                madakv_decode_attn call per layer and step (a layer needs the output of the layer below)
  op "window"   the prefill's own attention of the last window (madakv_window_attn_score), whose scores serve
                madakv_allocate and madakv_select_gather, then `steps` decode steps
  op "reevict"  as "evict", then madakv_reevict over all layers and one more decode step

Every pass starts with an eviction, which resets the cache: a pass can be repeated on the same state.  The outputs
are the scores, pooled scores, masses and counts of every head, the budgets and lengths, the decode outputs of every
step (which read every kept row of K and V; where a row lies in the reduced cache is the library's own affair: one
count that rounds the other way moves every later segment by a row) and, for "window", the attention output and
its log-sum-exp.

Inputs follow workloads.py: alternating text and image runs, Gaussian activations with a per-head modality
preference, heavy-hitter keys, a temperature per layer.
"""
import math

import torch

from paper_2506_15724_amd import binding as MB
from paper_2506_15724_amd import workloads as WL

DEV = "cuda:0"

# what a case has unless it says otherwise
BASE = dict(op="evict", n_layers=1, batch=1, n_q_heads=32, n_kv_heads=32, head_dim=128, ctx_len=16384, window=32,
            budget=2048, dtype="bf16", pool_k=7, steps=1, layers_per_call=1, out_fp32=1, cache_fp8=0, page_rows=0,
            n_modalities=2)


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    qwen = dict(n_layers=28, n_q_heads=28, n_kv_heads=4, ctx_len=32768, layers_per_call=28)
    long = dict(ctx_len=131072, window=64, budget=4096)
    return [
        # the smallest call: one layer of 8 short fp32 heads and a few tokens (a unit test, a toy model); launches and host
        _case("tiny_fp32", n_q_heads=8, n_kv_heads=8, head_dim=64, ctx_len=1024, window=16, budget=256, dtype="fp32",
              pool_k=1, steps=4),
        # one LLaVA-shaped layer of an ordinary prompt, scored by the prefill's own last-window attention
        _case("layer_8k_window", op="window", ctx_len=8192, budget=1024),
        # a prefill of four 16K prompts that evicts every layer as soon as it has been computed
        _case("prefill_16k_by_layer", n_layers=8, batch=4),
        # the same prompts with the whole model's prompt cache at hand: 32 layers in one call; the largest case
        _case("prefill_16k_model", n_layers=32, batch=4, layers_per_call=32),
        # grouped queries (7 per KV head, 224 proxy rows), 32K context, whole model
        _case("prefill_gqa_32k", **qwen),
        # a very long context, one layer, 64 proxy rows
        _case("prefill_128k", **long),
        # generation: most of the pass is decode, one call per layer and token
        _case("generate_16k", n_layers=8, batch=4, steps=24, layers_per_call=8, out_fp32=0),
        _case("generate_gqa_32k", **dict(qwen, steps=12, out_fp32=0)),
        _case("generate_128k_paged", **dict(long, steps=48, page_rows=64, out_fp32=0)),
        # the 8-bit reduced cache, which a user takes for its size
        _case("generate_16k_fp8", n_layers=8, batch=4, steps=24, layers_per_call=8, out_fp32=0, cache_fp8=1),
        # grouped queries scored by the prefill's last-window attention
        _case("window_gqa_32k", **dict(qwen, op="window", out_fp32=0)),
        # long generation: the cache is brought back to its size after some tokens
        _case("reevict_16k", op="reevict", n_layers=8, batch=4, steps=6, layers_per_call=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: head counts, dimensions, windows and options of the listed kinds, sizes over the whole range."""
    c = dict(BASE)
    c["op"] = rng.choice(["evict", "evict", "evict", "evict", "window", "reevict"])
    c["n_q_heads"], c["n_kv_heads"] = rng.choice([(32, 32), (32, 32), (28, 4), (8, 8), (32, 8), (12, 2), (20, 20)])
    c["head_dim"] = rng.choice([128, 128, 128, 64])
    group = c["n_q_heads"] // c["n_kv_heads"]
    c["window"] = rng.choice([w for w in (16, 32, 32, 40, 64) if w * group <= 256])
    if c["op"] == "evict" and group == 1 and rng.random() < 0.15:
        c["dtype"] = "fp32"
    most = 4096 if c["dtype"] == "fp32" else 32768 if c["op"] == "reevict" else 131072
    c["ctx_len"] = L = _log_int(rng, 700, most)
    c["budget"] = max(c["window"] + 24, int(L * math.exp(rng.uniform(math.log(1 / 32), math.log(1 / 3)))))
    c["n_layers"], c["batch"] = _log_int(rng, 1, 32), rng.choice([1, 1, 2, 4])
    size = 2 if c["dtype"] == "bf16" else 4
    while c["n_layers"] * c["batch"] * c["n_kv_heads"] * L * c["head_dim"] * size > 4 << 30:
        if c["batch"] > 1:
            c["batch"] //= 2
        else:
            c["n_layers"] = (c["n_layers"] + 1) // 2
    c["layers_per_call"] = c["n_layers"] if c["op"] == "reevict" else rng.choice([1, c["n_layers"]])
    c["steps"] = _log_int(rng, 1, 16)
    c["pool_k"] = rng.choice([1, 7, 7, 7, 5])
    c["out_fp32"] = rng.choice([0, 1])
    if c["dtype"] == "bf16":
        c["cache_fp8"] = rng.choice([0, 0, 0, 1])
        c["page_rows"] = rng.choice([0, 0, 0, 16, 64])
    c["n_modalities"] = rng.choice([2, 2, 2, 3])
    return c


def _workload(case, seed):
    L = case["ctx_len"]
    return WL.Workload(name="perf", n_layers=case["n_layers"], batch=case["batch"], n_q_heads=case["n_q_heads"],
                       n_kv_heads=case["n_kv_heads"], head_dim=case["head_dim"], ctx_len=L, window=case["window"],
                       budget=case["budget"], dtype=case["dtype"], pool_k=case["pool_k"], decode_steps=case["steps"],
                       image_tokens=(min(64, L // 16), min(1280, L // 4)), text_tokens=(min(16, L // 32), min(512, L // 8)),
                       n_images=0, heavy_hitters=0.01, bimodal_pref=False, cfg_id=seed, n_modalities=case["n_modalities"])


def prepare(case, seed):
    wl = _workload(case, seed)
    NL, B, Hq, H, d, L, W = (case[k] for k in ("n_layers", "batch", "n_q_heads", "n_kv_heads", "head_dim", "ctx_len", "window"))
    T, M, dt = case["steps"], case["n_modalities"], wl.torch_dtype
    masks = [WL.modality_mask(wl, b) for b in range(B)]
    mask = torch.stack([torch.from_numpy(m) for m in masks]).to(DEV)
    q = torch.empty(NL, B, Hq, W, d, dtype=dt, device=DEV)
    k = torch.empty(NL, B, H, L, d, dtype=dt, device=DEV)
    v = torch.empty(NL, B, H, L, d, dtype=dt, device=DEV)
    for l in range(NL):
        for b in range(B):
            q[l, b], k[l, b], v[l, b] = WL.layer_inputs(wl, l, b, masks[b], DEV)
    # a row of slack more than the steps for the step after a re-eviction
    eng = MB.MadaKV(n_layers=NL, batch=B, n_q_heads=Hq, n_kv_heads=H, head_dim=d, ctx_len=L, window=W, budget=case["budget"],
                    dtype=case["dtype"], pool_k=case["pool_k"], max_new_tokens=T + 1, out_fp32=case["out_fp32"],
                    n_modalities=M, cache_fp8=case["cache_fp8"], page_rows=case["page_rows"],
                    layers_per_call=case["layers_per_call"], device=DEV)
    extra = 1 if case["op"] == "reevict" else 0
    out = torch.empty(T + extra, NL, B, Hq, d, dtype=torch.float32 if case["out_fp32"] else dt, device=DEV)
    # one decode step's rows per layer, as the layers of a model hand them over
    steps = []
    for t in range(T + extra):
        dq, dk, dv = WL.decode_inputs_all(wl, t, DEV)
        steps.append([(dq[l:l + 1], dk[l:l + 1], dv[l:l + 1], out[t, l:l + 1]) for l in range(NL)])
    n = case["layers_per_call"]
    state = dict(case=case, eng=eng, mask=mask, steps=steps,
                 calls=[(l, min(n, NL - l), q[l:l + n], k[l:l + n], v[l:l + n]) for l in range(0, NL, n)])
    state["out"] = {"psi": eng.psi, "psi_pool": eng.psi_pool, "mass": eng.stats[..., :M].view(torch.float32),
                    "count": eng.stats[..., M:], "n_mod": eng.n_mod, "budgets": eng.budgets, "kv_len": eng.kv_len, "decode": out}
    if case["op"] == "window":
        odt = torch.float32 if case["out_fp32"] else dt
        state["attn"] = torch.empty(NL, B, Hq, W, d, dtype=odt, device=DEV)
        state["lse"] = torch.empty(NL, B, Hq, W, dtype=torch.float32, device=DEV)
        state["out"].update(attention=state["attn"], lse=state["lse"])
    if extra:
        # the queries of the last W tokens: the end of the prompt's window, then the generated ones
        made = torch.stack([torch.cat([layer[0] for layer in step]) for step in steps[:T]], dim=3)
        state["recent"] = torch.cat([q, made], dim=3)[:, :, :, -W:].contiguous()
    return state


def run(state):
    case, eng, mask = state["case"], state["eng"], state["mask"]
    for l, n, q, k, v in state["calls"]:
        if case["op"] == "window":
            eng.window_attn_score(l, n, q, k, v, mask, state["attn"][l:l + n], state["lse"][l:l + n])
            eng.allocate(l, n)
            eng.select_gather(l, n, k, v, mask)
        else:
            eng.evict(l, n, q, k, v, mask)
    for t in range(case["steps"]):
        for l, (q, k, v, out) in enumerate(state["steps"][t]):
            eng.decode_attn(l, 1, q, k, v, out)
    if case["op"] == "reevict":
        eng.reevict(0, case["n_layers"], state["recent"], mask)
        for l, (q, k, v, out) in enumerate(state["steps"][-1]):
            eng.decode_attn(l, 1, q, k, v, out)
    return state["out"]


def work(case):
    """Bytes: the prompt's K (for "window" V as well) and the queries read once, the scores written, the kept rows of V
    read, the reduced cache written, and read once per decode step.  Flops: the window's logits (for "window" the
    attention's second product too) and the decode steps' two products."""
    NL, B, Hq, H, d, L, W = (case[k] for k in ("n_layers", "batch", "n_q_heads", "n_kv_heads", "head_dim", "ctx_len", "window"))
    size = 2 if case["dtype"] == "bf16" else 4
    csize = 1 if case["cache_fp8"] else size
    heads, rows = NL * B * H, NL * B * H * min(case["budget"], L)        # a batch item keeps exactly its budget
    prompt = heads * L * d * size
    nbytes = prompt + NL * B * Hq * W * d * size + heads * L * 8 + B * L
    nbytes += rows * d * (size + 2 * csize) if case["op"] != "window" else prompt + rows * d * 2 * csize
    flops = 2 * NL * B * Hq * W * L * d * (2 if case["op"] == "window" else 1)
    steps = case["steps"] + (1 if case["op"] == "reevict" else 0)
    for t in range(steps):
        nbytes += (rows + heads * (t + 1)) * 2 * d * csize
        flops += 4 * NL * B * Hq * d * (rows // heads + t + 1)
    if case["op"] == "reevict":
        nbytes += (3 * rows + heads * case["steps"]) * d * csize          # the grown K read, the survivors' K and V moved at least in part
        flops += 2 * NL * B * Hq * W * d * (rows // heads + case["steps"])
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Measured over a dozen seeds per kind of case, the two scoring algorithms (one sweep, two sweeps: sums in another
    order) against each other and decode against a 64-bit attention over the same rows: scores within 7e-7 (2-norm) and
    6e-6 (largest), decode in fp32 within 8e-7 and 7e-6, in bf16 within 5e-5 and 3e-3 (one unit in the last place), up to
    5e-4 of the counts, budgets and lengths different by one (a mass that crosses theta one token earlier or later).
    The largest difference leaves room for a decode output whose head kept one other token of nearly equal score."""
    if case["out_fp32"] or case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 5e-3}
    return {"rel": 2e-4, "max": 1e-2, "differ": 5e-3}
