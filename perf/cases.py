"""The work whose speed counts, as cases: prefills of prompts with reused images, and the first-token head.

A prefill case is one prompt (or a packed batch of prompts) through a stack of decoder layers: one launch places
the reused image keys and values of all layers, then every layer runs through the chained layer call, as a serving
program does through paper_2512_12977_amd.runner.  Stacks have two to four layers of the model's true width (all
layers of a model are alike; a deeper bf16 stack would only let the roundings of two correct runs drift apart).
Weights, embeddings and cached K/V are random with the scales of the repository's synthetic workloads.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

import paper_2512_12977_amd as vlc
import vlc_synth as syn
from paper_2512_12977_amd import runner as R

# Expected price of a case in seconds, only to keep drawn cases below the largest listed one: rates that a plain
# implementation reaches.
_FLOP_RATE = {"bf16": 1.0e15, "f32": 2.0e13}
_BYTE_RATE = 4.0e12


def listed():
    def prefill(name, shape, layers, text_before, image_rows, image_cols, text_after, *, requests=1, images=1,
                image_step=0, text_between=0, plan="static", rate=10):
        """plan: "static" (rate = grid steps of 1/500 in every layer), "explicit" (rate = leading tokens of every
        image), "dynamic" (rate = mean rate in basis points, spread over the layers by the library's planner) or
        "all" (every row computed, nothing reused)."""
        return {"name": name, "kind": "prefill", "shape": shape, "layers": layers, "requests": requests,
                "text_before": text_before, "images": images, "image_rows": image_rows, "image_cols": image_cols,
                "image_step": image_step, "text_between": text_between, "text_after": text_after, "plan": plan,
                "rate": rate}

    return [
        # The smallest call: the tiny fp32 decoder with one 256-token image.  Latency, launches and host work.
        prefill("tiny_f32", "tiny", 2, 32, 16, 16, 16, plan="explicit", rate=13),
        # A short question about a cached image (the paper's prompts: little text, thousands of image tokens):
        # a hundred rows per layer, every weight read for them.
        prefill("question_7b", "7b", 4, 27, 37, 37, 43),
        # A system prompt and a question around one image: some 600 rows.
        prefill("prompt_7b", "7b", 4, 512, 32, 32, 64),
        # Four images between runs of text, other order than they were cached in, rates that fall with depth.
        prefill("images_7b", "7b", 4, 128, 36, 36, 128, images=4, text_between=128, plan="dynamic", rate=500),
        # The same with per-head norms and three-axis positions, images of unequal and odd sizes.
        prefill("images_q3_8b", "q3vl_8b", 4, 61, 29, 43, 87, images=3, image_step=5, text_between=33,
                plan="dynamic", rate=500),
        # The long-context batch of the throughput figure: 8 prompts of 18432 slots, 18944 rows per layer.
        prefill("batch_7b", "7b", 2, 100, 32, 32, 1948, requests=8, images=16),
        # A large model on a prompt of images and one question.
        prefill("images_72b", "72b", 2, 0, 36, 36, 256, images=8, plan="dynamic", rate=300),
        # First sight of an image: nothing can be reused, every row is computed (this fills the cache).
        prefill("first_sight_7b", "7b", 2, 128, 36, 36, 128, images=4, text_between=128, plan="all", rate=500),
        # Mixture of experts: a question (about a hundred rows, few per expert), the prompt of some 600 rows
        # (forty per expert), and a batch.
        prefill("question_moe", "q3vl_30b_a3b", 3, 27, 37, 37, 43),
        prefill("prompt_moe", "q3vl_30b_a3b", 3, 512, 32, 32, 64),
        prefill("batch_moe", "q3vl_30b_a3b", 2, 100, 32, 32, 924, requests=6, images=8),
        # The first token of every prompt of a batch: final norm, output matrix, greedy choice.
        {"name": "head_7b", "kind": "head", "shape": "7b", "requests": 8, "rows": 2368},
    ]


def _log(rng, lo, hi):
    """A whole number spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(_price(c) for c in listed())
    while True:
        if rng.random() < 0.1:
            return {"kind": "head", "shape": rng.choice(["7b", "q3vl_8b", "72b", "q3vl_30b_a3b"]),
                    "requests": _log(rng, 1, 64), "rows": _log(rng, 64, 8192)}
        shape = rng.choice(["tiny", "tiny_bias", "tiny_q3", "tiny_moe", "7b", "7b", "7b", "7b", "q3vl_8b", "q3vl_8b",
                            "72b", "q3vl_30b_a3b", "q3vl_30b_a3b"])
        tiny = shape.startswith("tiny")
        # a short question, a prompt, or long text; one request in most cases
        c = {"kind": "prefill", "shape": shape, "layers": 2,
             "requests": 1 if rng.random() < 0.6 else rng.randint(2, 8), "text_before": rng.randint(0, 64),
             "images": 1 if rng.random() < 0.4 else rng.randint(2, 16), "image_rows": rng.randint(8, 40),
             "image_cols": rng.randint(8, 40), "image_step": rng.choice([0, 0, 1, 3]),
             "text_between": rng.choice([0, 0, _log(rng, 1, 128)]), "text_after": _log(rng, 8, 1024),
             "plan": rng.choice(["static", "static", "dynamic"]), "rate": 0}
        if tiny:
            c.update(requests=rng.randint(1, 2), images=rng.randint(1, 2), text_after=_log(rng, 8, 128),
                     image_rows=rng.randint(4, 20), image_cols=rng.randint(4, 20))
        c["rate"] = rng.randint(5, 30) if c["plan"] == "static" else rng.randint(100, 600)
        if rng.random() < 0.1:
            c["plan"], c["rate"] = "all", 500
        if _price(c) <= most and _state_bytes(c) <= 60e9:
            return c


# ---------------------------------------------------------------------------------------------------------------
# what a case describes
# ---------------------------------------------------------------------------------------------------------------
def _shape(case):
    sh = syn.SHAPES[case["shape"]]
    return dataclasses.replace(sh, L=case["layers"]) if case["kind"] == "prefill" else sh


def _requests(case):
    """The packed requests and the number of rows of the cached-image pool.  All requests of a batch ask about the
    same images, the text before and after them split differently; images are used in reversed order, so the
    position shifts have both signs."""
    sizes = [(case["image_rows"], case["image_cols"] + i * case["image_step"]) for i in range(case["images"])]
    grid_ids = bool(_shape(case).mrope_section)
    pool_row, old_pos, rows, at = [], [], 0, 0
    for r, c in sizes:
        pool_row.append(rows)
        old_pos.append(at)
        rows += r * c
        at += max(r, c) if grid_ids else r * c
    requests, first = [], 0
    for b in range(case["requests"]):
        before = case["text_before"] + (37 * b) % (case["text_after"] // 2 + 1)
        after = case["text_before"] + case["text_after"] - before
        parts = [("text", before)] if before else []
        for k, i in enumerate(reversed(range(len(sizes)))):
            if k and case["text_between"]:
                parts.append(("text", case["text_between"]))
            parts.append(("image", sizes[i][0], sizes[i][1], old_pos[i], pool_row[i]))
        parts.append(("text", after))
        segments, s = [], 0
        for p in parts:
            n = p[1] if p[0] == "text" else p[1] * p[2]
            segments.append(syn.Segment(s, n, False) if p[0] == "text" else syn.Segment(s, n, True, p[3], p[4]))
            s += n
        pos3 = syn.grid_positions([p[:3] for p in parts]) if grid_ids else None
        requests.append(syn.Request(segments, first, 0, pos3))
        first += s
    return requests, rows


def _rates(case):
    """(grid step per layer or None, leading tokens per layer or None)"""
    L = case["layers"]
    if case["plan"] == "explicit":
        return None, np.full(L, case["rate"], dtype=np.int32)
    if case["plan"] == "dynamic":
        return vlc.vlc_plan_layer_rates(syn.sensitivity_table(L, 150, 1), vlc.vlc_plan_budget_steps(case["rate"], L)), None
    return np.full(L, case["rate"], dtype=np.int32), None


def _rows(case):
    """Per layer: (rows computed, (row, visible key) pairs, image tokens reused); and the slots of the batch."""
    requests, _ = _requests(case)
    k, counts = _rates(case)
    per_layer = []
    for l in range(case["layers"]):
        n = pairs = reused = 0
        for r in requests:
            for s in r.segments:
                take = s.length
                if s.is_image:
                    take = min(s.length, int(counts[l])) if counts is not None else int(k[l]) * s.length // 500
                    reused += s.length - take
                n += take
                pairs += take * s.start + take * (take + 1) // 2
        per_layer.append((n, pairs, reused))
    return per_layer, sum(r.S for r in requests)


def _layer_elems(sh):
    """Weight elements of a layer, and of them those that every row multiplies."""
    attn = sh.n_qkv * sh.H + sh.H * sh.Hq * sh.D
    mlp = 3 * sh.H * sh.I
    if sh.n_experts:
        return attn + sh.n_experts * (mlp + sh.H), attn + sh.top_k * mlp + sh.n_experts * sh.H
    return attn + mlp, attn + mlp


def work(case):
    """Weights, first hidden rows and reused K/V read once, K/V caches and last hidden rows written once; the
    products of the rows that are computed (each with its own experts only) and their attention over what they see."""
    sh = _shape(case)
    e = 2 if sh.dtype == "bf16" else 4
    if case["kind"] == "head":
        n = case["requests"]
        return {"bytes": sh.vocab * sh.H * e + n * (sh.H * e + sh.vocab * 4), "flops": 2.0 * n * sh.vocab * sh.H}
    layers, slots = _rows(case)
    held, used = _layer_elems(sh)
    kv = 2 * sh.Hkv * sh.D * e
    nbytes = (layers[0][0] + layers[-1][0]) * sh.H * e
    flops = 0.0
    for n, pairs, reused in layers:
        weights = held
        if sh.n_experts:   # with few rows not every expert is chosen: the expected share, every choice alike
            hit = sh.n_experts * (1.0 - (1.0 - sh.top_k / sh.n_experts) ** n)
            weights = held - (sh.n_experts - hit) * 3 * sh.H * sh.I
        nbytes += weights * e + reused * kv + slots * kv
        flops += 2.0 * n * used + 4.0 * pairs * sh.Hq * sh.D
    return {"bytes": float(nbytes), "flops": flops}


def _price(case):
    w = work(case)
    return w["flops"] / _FLOP_RATE[_shape(case).dtype] + w["bytes"] / _BYTE_RATE


def _state_bytes(case):
    sh = _shape(case)
    if case["kind"] == "head":
        return 2.0 * sh.vocab * sh.H
    layers, slots = _rows(case)
    return case["layers"] * (2.0 * _layer_elems(sh)[0] + 8.0 * slots * sh.Hkv * sh.D) + slots * sh.H * 2.0 + \
        layers[0][0] * (6.0 * sh.n_qkv + 12.0 * sh.H + 2.0 * sh.I * max(1, sh.top_k) + 2.0 * sh.H * sh.top_k)


def tolerance(case):
    """About four times what this path differs by from itself with the sums of its products and of its attention
    taken in another order (no k ranges, no key shares, other tiles): fp32 3e-7; dense bf16 stacks 0.2-0.6 % after
    two layers and 1 % after four, with single elements off by 6 % of the rms (one flipped rounding moves every
    later value of its row); expert stacks, whose projections into the residual stream are scaled down, 0.1 %.
    Scores of the head differ by one rounding of a normed row's element at most."""
    sh = _shape(case)
    if sh.dtype == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    if case["kind"] == "head":
        return {"rel": 1e-4}
    if sh.n_experts:
        return {"rel": 0.005, "max": 0.25}
    return {"rel": 0.025 if case["layers"] <= 2 else 0.03, "max": 0.25}


# ---------------------------------------------------------------------------------------------------------------
# a user's program
# ---------------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    sh = _shape(case)
    dt = R.torch_dtype(sh.dtype)
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(seed)

    def normal(*size, scale=1.0, mean=0.0):
        t = torch.empty(size, device=dev, dtype=torch.float32).normal_(mean, scale, generator=g)
        return t if dt == torch.float32 else t.to(dt)

    if case["kind"] == "head":
        n = case["requests"]
        code = vlc.VLC_BF16 if sh.dtype == "bf16" else vlc.VLC_F32
        return {"kind": "head", "eps": sh.eps, "h": normal(case["rows"], sh.H), "w_norm": normal(sh.H, scale=0.02, mean=1.0),
                "w_out": normal(sh.vocab, sh.H, scale=0.02),
                "rows": torch.randint(0, case["rows"], (n,), generator=g, device=dev, dtype=torch.int32),
                "logits": torch.empty((n, sh.vocab), device=dev, dtype=torch.float32),
                "token": torch.empty((n,), device=dev, dtype=torch.int32),
                "ws": torch.empty(vlc.vlc_first_token_workspace_bytes(sh.H, n, code), device=dev, dtype=torch.uint8)}

    requests, pool_rows = _requests(case)
    k, counts = _rates(case)
    plans = R.DevicePlans(requests, sh.L, k=k, count_override=counts, all_rows=case["plan"] == "all")
    slots, L = plans.total_slots, sh.L
    weights = [R.DeviceWeights.random(sh, dt, seed * 131 + l) for l in range(L)]
    # text rows are small against image rows, as in the synthetic workloads
    h0 = normal(slots, sh.H)
    for r in requests:
        for s in r.segments:
            if not s.is_image:
                h0[r.kv_start + s.start:r.kv_start + s.start + s.length] *= sh.text_scale
    k_pool = [normal(pool_rows, sh.Hkv, sh.D) for _ in range(L)]
    v_pool = [normal(pool_rows, sh.Hkv, sh.D) for _ in range(L)]
    k_cache = [torch.zeros((slots, sh.Hkv, sh.D), device=dev, dtype=dt) for _ in range(L)]
    v_cache = [torch.zeros((slots, sh.Hkv, sh.D), device=dev, dtype=dt) for _ in range(L)]
    shape_rec = R.make_shape(sh)
    n_in = [slots] + plans.n_rows[:-1]
    return {"kind": "prefill", "shape": shape_rec, "base": sh.rope_base, "weights": weights, "plans": plans,
            "records": [plans.record(l, n_in[l], slots) for l in range(L)],
            "shift": R.ShiftJobs(plans, k_pool, v_pool, k_cache, v_cache), "h0": h0,
            "hbuf": [torch.empty((max(plans.n_rows), sh.H), device=dev, dtype=dt) for _ in range(2)],
            "k_cache": k_cache, "v_cache": v_cache, "ws": R.Workspace(shape_rec, max(plans.n_rows))}


def run(state):
    s = state
    if s["kind"] == "head":
        vlc.vlc_first_token(s["h"], s["rows"], s["eps"], s["w_norm"], s["w_out"], s["logits"], s["token"], s["ws"])
        return {"logits": s["logits"], "token": s["token"]}
    s["shift"].run(s["base"])
    h = R.run_layers(s["shape"], s["weights"], s["plans"], s["records"], s["h0"], s["hbuf"], s["k_cache"],
                     s["v_cache"], s["ws"])
    return {"h": h[:s["plans"].n_rows[-1]], "k": s["k_cache"], "v": s["v_cache"]}
