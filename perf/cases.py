"""Performance cases of the FlashBlock attention path on one GPU: what a block-diffusion program asks of the library.

A case is one whole piece of a denoising loop through the public binding: a block of diffusion steps (a refresh step
that streams the prefix cache, then reuse steps that read only the cached partial), a single reuse step, a head-wise
selective refresh, or a sparse block with its key-block selection.  The raw cached partial (o, m) is not an output:
its reference m is the implementation's choice by contract.  Its log-normaliser is, and every case that refreshes a
partial also takes at least one step that reads it, so what was cached shows in that step's output.
"""
import math

import torch

from paper_2602_05305_amd import flashblock as fb

DEV = "cuda"
TORCH_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
STEP_SIGMA = 0.05      # a block's queries, keys and values drift from step to step


def _case(kind, dtype, batch, heads, head_dim, prefix, block, steps, **more):
    """heads: "query/kv"."""
    hq, hkv = (int(x) for x in heads.split("/"))
    return {"kind": kind, "dtype": dtype, "batch": batch, "n_q_heads": hq, "n_kv_heads": hkv, "head_dim": head_dim,
            "prefix_len": prefix, "block_len": block, "steps": steps, **more}


def listed():
    """Sizes are the repository's benchmark configurations and tests, or generic neighbours of them."""
    cases = {
        # one reuse step of one layer of a language model: the call made most often, 7 of 8 steps
        "reuse_llm": _case("reuse", "bf16", 1, "32/8", 128, 2048, 32, 1),
        # fp32 storage at its smallest: a whole block of 4 steps, launch latency throughout
        "tiny_f32_block": _case("dense", "f32", 1, "4/4", 64, 256, 16, 4),
        # fp32 storage at a model's head layout and a short ragged context: checking a model in full precision
        "f32_4k_block": _case("dense", "f32", 1, "32/8", 128, 4111, 32, 2),
        # the headline: a block of 8 steps, refreshed once, over a 32K context
        "llm_32k_block": _case("dense", "bf16", 1, "32/8", 128, 32768, 32, 8),
        # long context: the refresh step dominates
        "long_128k_block": _case("dense", "bf16", 1, "32/8", 128, 131072, 32, 2),
        # a batch of medium, ragged contexts of a small model (head_dim 64), offline generation
        "batch_d64_block": _case("dense", "bf16", 16, "16/4", 64, 5003, 24, 4),
        # serving with a paged cache: 32 sequences of unequal length, blocks of 32
        "paged_b32_block": _case("paged", "bf16", 32, "32/8", 128, 8192, 32, 2, min_len=512, page=256),
        # serving at the largest batch, small blocks
        "paged_b128_block": _case("paged", "bf16", 128, "32/8", 128, 12288, 4, 2, min_len=512, page=256),
        # video: block of 3 latent frames, prefix of 8 blocks, refresh and one reuse step (matrix-bound)
        "video_block": _case("dense", "bf16", 1, "12/12", 128, 37440, 4680, 2),
        # video: the reuse step by itself
        "video_reuse": _case("reuse", "bf16", 1, "12/12", 128, 4680, 4680, 1),
        # video, head-wise selective reuse: 3 of 12 heads are refreshed, the others keep their cached partial
        "video_heads": _case("heads", "bf16", 1, "12/12", 128, 37440, 4680, 1, active=3),
        # sparse attention with residual reuse: pooling, top-k selection, refresh, three reuse steps
        "sparse_64k_block": _case("sparse", "bf16", 1, "32/8", 128, 65536, 32, 4, key_block=64, topk=256),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["dense", "dense", "dense_f32", "paged", "paged", "video", "heads", "reuse", "sparse", "sparse"])
    hkv = rng.choice([2, 4, 8])
    heads = "%d/%d" % (hkv * rng.choice([1, 2, 4, 4, 8]), hkv)
    d = rng.choice([64, 128, 128])
    steps = rng.randint(2, 8)
    while True:
        if kind == "dense":
            c = _case("dense", "bf16", _log_int(rng, 1, 16), heads, d, _log_int(rng, 500, 131072), rng.randint(1, 64), steps)
        elif kind == "dense_f32":
            c = _case("dense", "f32", rng.randint(1, 2), heads, d, _log_int(rng, 100, 6000), rng.randint(4, 48), steps)
        elif kind == "paged":
            hi = _log_int(rng, 700, 12288)
            c = _case("paged", "bf16", _log_int(rng, 4, 128), heads, d, hi, rng.choice([4, 8, 16, 32, rng.randint(1, 32)]),
                      rng.randint(2, 4), min_len=rng.randint(1, hi // 2), page=rng.choice([64, 128, 256]))
        elif kind in ("video", "heads"):
            h = rng.randint(4, 12)
            c = _case("dense" if kind == "video" else "heads", "bf16", 1, "%d/%d" % (h, h), rng.choice([64, 128, 128]),
                      _log_int(rng, 3000, 37440), rng.randint(1000, 4680), 2 if kind == "video" else 1)
            if kind == "heads":
                c["active"] = rng.randint(1, h - 1)
        elif kind == "reuse":
            block = _log_int(rng, 4, 4680)
            if block > 1000:
                heads = "%d/%d" % (hkv, hkv)
            c = _case("reuse", "bf16", _log_int(rng, 1, 16) if block <= 64 else 1, heads, d, _log_int(rng, 500, 4680), block, 1)
        else:
            key_block = rng.choice([64, 64, 128])
            prefix = _log_int(rng, 8192, 131072)
            c = _case("sparse", "bf16", rng.randint(1, 2), heads, d, prefix, rng.randint(4, 32), steps, key_block=key_block,
                      topk=max(1, int(rng.uniform(0.1, 0.5) * prefix / key_block)), rule=rng.choice(["pooled", "mass"]))
        w = work(c)
        if w["bytes"] <= 2.2e9 and w["flops"] <= 1.1e12:
            return c


# ---------------------------------------------------------------------------------------------- inputs
def _lens(c):
    """Prefix length of every sequence of a paged batch, shortest first: spread evenly over [min_len, prefix_len]."""
    n = c["batch"]
    return [c["min_len"] + (c["prefix_len"] - c["min_len"]) * i // max(1, n - 1) for i in range(n)]


def _inputs(c, seed):
    """Everything that is drawn, from the seed alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    dt = TORCH_DTYPE[c["dtype"]]
    B, Hq, Hkv, d, P, Bq = (c[k] for k in ("batch", "n_q_heads", "n_kv_heads", "head_dim", "prefix_len", "block_len"))

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=dt)

    x = {}
    if c["kind"] == "paged":
        page = c["page"]
        order = torch.randperm(B, generator=g, device=DEV)
        lens = torch.tensor(_lens(c), device=DEV, dtype=torch.int32)[order].contiguous()
        need = [-(-n // page) for n in lens.tolist()]
        pages = sum(need) + 3
        ids = torch.randperm(pages, generator=g, device=DEV).tolist()
        table = torch.full((B, -(-P // page)), -1, dtype=torch.int32)
        at = 0
        for b, n in enumerate(need):
            table[b, :n] = torch.tensor(ids[at:at + n], dtype=torch.int32)
            at += n
        x["lens"], x["table"] = lens, table.to(DEV)
        x["k"], x["v"] = normal(pages, Hkv, page, d), normal(pages, Hkv, page, d)
    else:
        x["k"], x["v"] = normal(B, Hkv, P, d), normal(B, Hkv, P, d)
    if c["kind"] in ("reuse", "heads"):
        x["q_before"] = normal(B, Hq, Bq, d)          # the query the cached partial was computed with
    if c["kind"] == "heads":
        on = torch.zeros(B * Hq, dtype=torch.uint8, device=DEV)
        on[torch.randperm(Hq, generator=g, device=DEV)[:c["active"]]] = 1
        x["head_mask"] = on.view(B, Hq)
    q, kb, vb = normal(B, Hq, Bq, d), normal(B, Hkv, Bq, d), normal(B, Hkv, Bq, d)
    x["steps"] = [(q, kb, vb)]
    for _ in range(1, c["steps"]):
        q, kb, vb = (t + STEP_SIGMA * normal(*t.shape) for t in (q, kb, vb))
        x["steps"].append((q, kb, vb))
    return x


def prepare(c, seed):
    """Inputs, the caller-owned buffers (cached partial, workspace, outputs) and the shape descriptor."""
    x = _inputs(c, seed)
    B, Hq, Hkv, d, P, Bq = (c[k] for k in ("batch", "n_q_heads", "n_kv_heads", "head_dim", "prefix_len", "block_len"))
    shape = fb.make_shape(B, Hq, Hkv, d, Bq, P, c["dtype"])

    def floats(*dims):
        return torch.zeros(dims, device=DEV, dtype=torch.float32)

    def bytes_(n):
        return torch.empty(n, device=DEV, dtype=torch.uint8)

    s = dict(x, case=c, shape=shape, o=floats(B, Hq, Bq, d), m=floats(B, Hq, Bq), lse=floats(B, Hq, Bq),
             outs=[torch.zeros_like(q) for q, _, _ in x["steps"]])
    if c["kind"] == "dense":
        s["ws"] = bytes_(fb.fb_workspace_bytes(shape))
    elif c["kind"] == "paged":
        s["kv"] = fb.make_paged_kv(x["k"], x["v"], x["table"], x["lens"])
        s["ws"] = bytes_(fb.fb_workspace_bytes(shape, 0, 0, fb.fb_paged_splits(shape)))
    elif c["kind"] in ("reuse", "heads"):
        s["ws"] = bytes_(fb.fb_workspace_bytes(shape))
        s["lse_out"] = floats(B, Hq, Bq)
        fb.fb_external_partial(shape, x["q_before"], x["k"], x["v"], s["o"], s["m"], s["lse"], s["ws"])
        if c["kind"] == "heads":
            s["ws"] = bytes_(fb.fb_workspace_bytes(shape, 0, 0, fb.fb_external_heads_splits(shape, c["active"])))
    else:
        kb = c["key_block"]
        s["ws"] = bytes_(fb.fb_workspace_bytes(shape, kb, c["topk"]))
        if _mass(c):
            s["sel_ws"] = bytes_(fb.fb_select_mass_workspace_bytes(shape, kb))
        else:
            s["sel_ws"] = bytes_(fb.fb_select_workspace_bytes(shape, kb))
            s["pooled"] = floats(B, Hkv, -(-P // kb), d)
        s["sel"] = torch.zeros((B, Hq, c["topk"]), device=DEV, dtype=torch.int32)
        s["res"] = (floats(B, Hq, Bq, d), floats(B, Hq, Bq), floats(B, Hq, Bq))
    return s


def _mass(c):
    return c.get("rule", "pooled") == "mass"


# ---------------------------------------------------------------------------------------------- the pass
def run(s):
    c, shape, o, m, lse, outs = s["case"], s["shape"], s["o"], s["m"], s["lse"], s["outs"]
    kind = c["kind"]
    if kind == "reuse":
        q, kb, vb = s["steps"][0]
        fb.fb_internal_merge(shape, q, kb, vb, o, m, lse, outs[0], s["lse_out"])
        return {"out": outs[0], "lse": s["lse_out"]}
    if kind == "heads":
        q, kb, vb = s["steps"][0]
        fb.fb_external_partial_heads(shape, q, s["k"], s["v"], s["head_mask"], o, m, lse, s["ws"], c["active"])
        fb.fb_internal_merge(shape, q, kb, vb, o, m, lse, outs[0], s["lse_out"])
        return {"out": outs[0], "lse": s["lse_out"], "lse_part": lse}
    if kind == "sparse":
        return _run_sparse(s)
    for t, (q, kb, vb) in enumerate(s["steps"]):
        if t > 0:
            fb.fb_internal_merge(shape, q, kb, vb, o, m, lse, outs[t])
        elif kind == "paged":
            fb.fb_refresh_step_paged(shape, q, s["kv"], kb, vb, o, m, lse, outs[t], None, s["ws"])
        else:
            fb.fb_refresh_step(shape, q, s["k"], s["v"], kb, vb, o, m, lse, outs[t], None, s["ws"])
    return {"out": outs, "lse_part": lse}


def _run_sparse(s):
    c, shape, o, m, lse, outs, res = s["case"], s["shape"], s["o"], s["m"], s["lse"], s["outs"], s["res"]
    key_block, topk = c["key_block"], c["topk"]
    q0 = s["steps"][0][0]
    if _mass(c):      # the mask comes from full attention at the block's first step
        fb.fb_external_partial(shape, q0, s["k"], s["v"], o, m, lse, s["ws"])
        fb.fb_select_topk_mass(shape, q0, s["k"], lse, key_block, topk, s["sel"], None, s["sel_ws"])
    else:
        fb.fb_pool_keys(shape, s["k"], key_block, s["pooled"])
        fb.fb_select_topk(shape, q0, s["pooled"], key_block, topk, s["sel"], s["sel_ws"])
    for t, (q, kb, vb) in enumerate(s["steps"]):
        mode = fb.FB_SPARSE_REFRESH if t == 0 else fb.FB_SPARSE_REUSE_SAME_SELECTION
        fb.fb_sparse_external_residual(shape, mode, q, s["k"], s["v"], key_block, topk, s["sel"], *res, o, m, lse, s["ws"])
        fb.fb_internal_merge(shape, q, kb, vb, o, m, lse, outs[t])
    return {"out": outs, "lse_part": lse, "res_lse": res[2], "sel": s["sel"]}


# ---------------------------------------------------------------------------------------------- what it has to do
def work(c):
    B, Hq, Hkv, d, P, Bq = (c[k] for k in ("batch", "n_q_heads", "n_kv_heads", "head_dim", "prefix_len", "block_len"))
    e = 4 if c["dtype"] == "f32" else 2
    rows = B * Hq * Bq
    partial = rows * (d + 2) * 4
    block = (2 * rows * d + 2 * B * Hkv * Bq * d) * e            # q, out, block K and V of one step
    block_flops = 4 * rows * Bq * d
    prefix = 2 * B * Hkv * P * d * e
    prefix_flops = 4 * rows * P * d
    if c["kind"] == "paged":
        total = sum(_lens(c))
        prefix, prefix_flops = 2 * Hkv * total * d * e, 4 * Hq * Bq * total * d
    steps = c["steps"]
    if c["kind"] == "reuse":
        return {"bytes": block + partial + rows * 4, "flops": block_flops}
    if c["kind"] == "heads":
        a = c["active"] / Hq
        return {"bytes": a * (prefix + partial) + block + partial + rows * 4, "flops": a * prefix_flops + block_flops}
    if c["kind"] == "sparse":
        # selection reads K once more (its arithmetic is small or, by mass, the score product), a reuse step reads the
        # key blocks that any head of a KV group selected (independent choices) and computes each head's own
        density = min(1.0, c["topk"] * c["key_block"] / P)
        union = 1 - (1 - density) ** (Hq // Hkv)
        bytes_ = 1.5 * prefix + (prefix if _mass(c) else 0) + 2 * partial + steps * (block + partial)
        bytes_ += (steps - 1) * (union * prefix + 2 * partial) + B * Hq * c["topk"] * 4
        flops = prefix_flops * (1 + (1.5 if _mass(c) else 0) + (steps - 1) * density) + steps * block_flops
        return {"bytes": bytes_, "flops": flops}
    return {"bytes": prefix + partial + steps * block + (steps - 1) * partial, "flops": prefix_flops + steps * block_flops}


def tolerance(c):
    if c["dtype"] == "f32":
        return {"rel": 5e-6, "max": 5e-5}        # against 64 bits: 3e-7 to 9e-7
    if c["kind"] == "sparse":
        # a tie in the selection's fp32 scores swaps two key blocks of one head and shifts the ascending list between them
        return {"rel": 1e-2, "max": 0.1, "differ": 0.05}
    return {"rel": 1e-2, "max": 2e-2}            # against 64 bits: 2.3e-3, the rounding of weights and outputs to bf16


# ---------------------------------------------------------------------------------------------- the same in 64 bits
def _attend(q, k, v, scale):
    """(exp-sum-normalised output, log-normaliser) of q [R,d] against k, v [n,d] in 64 bits, a slab of rows at a time."""
    outs, lses = [], []
    kt = k.t().contiguous()
    slab = max(1, (1 << 27) // max(1, k.shape[0]))
    for r0 in range(0, q.shape[0], slab):
        s = (q[r0:r0 + slab] @ kt) * scale
        lse = torch.logsumexp(s, 1)
        s.sub_(lse[:, None]).exp_()
        outs.append(s @ v)
        lses.append(lse)
    return torch.cat(outs), torch.cat(lses)


def _external(c, x, q):
    """Full attention of q over the prefix: A [B,Hq,Bq,d], L [B,Hq,Bq]."""
    A = torch.empty(q.shape, device=DEV, dtype=torch.float64)
    L = torch.empty(q.shape[:3], device=DEV, dtype=torch.float64)
    G, scale = c["n_q_heads"] // c["n_kv_heads"], 1 / math.sqrt(c["head_dim"])
    for b in range(c["batch"]):
        for h in range(c["n_kv_heads"]):
            k, v = _prefix(c, x, b, h)
            heads = slice(h * G, (h + 1) * G)
            a, l = _attend(q[b, heads].reshape(-1, q.shape[3]).double(), k, v, scale)
            A[b, heads], L[b, heads] = a.view(A[b, heads].shape), l.view(L[b, heads].shape)
    return A, L


def _prefix(c, x, b, h):
    if c["kind"] != "paged":
        return x["k"][b, h].double(), x["v"][b, h].double()
    n, page, d = int(x["lens"][b]), c["page"], c["head_dim"]
    ids = x["table"][b, :-(-n // page)].long()
    return tuple(t[ids, h].reshape(-1, d)[:n].double() for t in (x["k"], x["v"]))


def _merge(c, A, L, step):
    """Block-internal attention of a step composed with the external (A, L): output and log-normaliser."""
    q, kb, vb = (t.double() for t in step)
    G, scale = c["n_q_heads"] // c["n_kv_heads"], 1 / math.sqrt(c["head_dim"])
    out, lse = torch.empty_like(A), torch.empty_like(L)
    for b in range(c["batch"]):
        for h in range(c["n_kv_heads"]):
            heads = slice(h * G, (h + 1) * G)
            a, l = _attend(q[b, heads].reshape(-1, q.shape[3]), kb[b, h], vb[b, h], scale)
            a, l = a.view(A[b, heads].shape), l.view(L[b, heads].shape)
            both = torch.logaddexp(l, L[b, heads])
            out[b, heads] = a * (l - both).exp()[..., None] + A[b, heads] * (L[b, heads] - both).exp()[..., None]
            lse[b, heads] = both
    return out, lse


def _exact_sparse(c, x):
    G, scale, kb = c["n_q_heads"] // c["n_kv_heads"], 1 / math.sqrt(c["head_dim"]), c["key_block"]
    B, Hq, Bq, P, d = (c[k] for k in ("batch", "n_q_heads", "block_len", "prefix_len", "head_dim"))
    nblk = -(-P // kb)
    block_of = torch.arange(P, device=DEV) // kb
    counts = torch.bincount(block_of, minlength=nblk).double()
    steps = x["steps"]
    A = [torch.empty((B, Hq, Bq, d), device=DEV, dtype=torch.float64) for _ in steps]
    L = [torch.empty((B, Hq, Bq), device=DEV, dtype=torch.float64) for _ in steps]
    sel = torch.empty((B, Hq, c["topk"]), device=DEV, dtype=torch.int32)
    res_lse = torch.empty((B, Hq, Bq), device=DEV, dtype=torch.float64)
    for b in range(B):
        for h in range(Hq):
            k, v = x["k"][b, h // G].double(), x["v"][b, h // G].double()
            q0 = steps[0][0][b, h].double()
            if _mass(c):
                p = torch.softmax((q0 @ k.t().contiguous()) * scale, 1).mean(0)
                score = torch.zeros(nblk, device=DEV, dtype=torch.float64).index_add_(0, block_of, p)
            else:
                pooled = torch.zeros((nblk, d), device=DEV, dtype=torch.float64).index_add_(0, block_of, k) / counts[:, None]
                score = pooled @ q0.mean(0)
            chosen = torch.topk(score, c["topk"]).indices.sort().values
            sel[b, h] = chosen.int()
            on = torch.zeros(nblk, device=DEV, dtype=torch.bool)
            on[chosen] = True
            on = on[block_of]
            a_res, l_res = _attend(q0, k[~on], v[~on], scale)
            res_lse[b, h] = l_res
            ks, vs = k[on], v[on]
            for t, (q, _, _) in enumerate(steps):
                a, l = _attend(q[b, h].double(), ks, vs, scale)
                both = torch.logaddexp(l, l_res)
                A[t][b, h] = a * (l - both).exp()[:, None] + a_res * (l_res - both).exp()[:, None]
                L[t][b, h] = both
    outs = [_merge(c, A[t], L[t], step)[0] for t, step in enumerate(steps)]
    return {"out": outs, "lse_part": L[-1], "res_lse": res_lse, "sel": sel}


def exact(c, seed):
    x = _inputs(c, seed)
    if c["kind"] == "sparse":
        return _exact_sparse(c, x)
    if c["kind"] == "reuse":
        out, lse = _merge(c, *_external(c, x, x["q_before"]), x["steps"][0])
        return {"out": out, "lse": lse}
    if c["kind"] == "heads":
        A, L = _external(c, x, x["q_before"])
        A1, L1 = _external(c, x, x["steps"][0][0])
        on = x["head_mask"].bool()
        A[on], L[on] = A1[on], L1[on]
        out, lse = _merge(c, A, L, x["steps"][0])
        return {"out": out, "lse": lse, "lse_part": L}
    A, L = _external(c, x, x["steps"][0][0])
    return {"out": [_merge(c, A, L, step)[0] for step in x["steps"]], "lse_part": L}
