"""The work that a program using this package has it do, as measurable cases.

A case is one call, or one short sequence of calls, of a serving loop with speculative decoding: a transformer
layer's verification attention (with the cache append in front of it), the accept step in its modes, the early-exit
check with pruning and restore, the whole one-shot step, the chunked (frontier) step.  Sizes are those of the
package's own workload table (``workloads.CONFIGS``), of its tests, or lie between them.

``listed()`` gives the fixed cases, ``draw(rng)`` one more case of the same ranges, ``prepare(case, seed)`` what the
program holds on the GPU before the call, ``run(state)`` one pass, ``work(case)`` the bytes and operations a pass
cannot do without, ``tolerance(case)`` how far another correct implementation may be off and ``exact(case, seed)`` the
result in 64 bits by plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2604_20503_amd as fsr
from paper_2604_20503_amd import binding
from paper_2604_20503_amd.frontier import ChunkedVerifier

PAGE = 16
RANK_K = 10          # early exit: a draft survives while fewer than K scores exceed its own
KV8_SCALE = 0.02     # 8-bit caches: value of one unit of the E4M3 code (N(0, 1) keys and values use its whole range)
ALPHA = 0.78         # acceptance per draft of the synthetic distributions, for the bytes an accept step needs
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


# ---------------------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # one user's decode step, the smallest call there is: append one layer's rows, attend over a short context
        dict(name="layer_b1", kind="layer", B=1, H_q=32, H_kv=8, D=128, dtype="bf16", layout="head", ctx="uniform",
             ctx_lo=257, ctx_hi=257, spec_lo=3, spec_hi=3, layers=1, plan=False, lengths=1),
        # fp32 heads of 64 on a handful of requests (workload 1: small draft-sized models, debugging at full precision)
        dict(name="attn_f32_d64_b4", kind="attn", B=4, H_q=8, H_kv=2, D=64, dtype="f32", layout="head", ctx="uniform",
             ctx_lo=64, ctx_hi=256, spec_lo=0, spec_hi=4, layers=1, plan=False, lengths=2),
        # heads of 64 at an ordinary batch (small target models)
        dict(name="attn_d64_b32", kind="attn", B=32, H_q=32, H_kv=8, D=64, dtype="bf16", layout="head", ctx="uniform",
             ctx_lo=256, ctx_hi=4096, spec_lo=1, spec_hi=8, layers=1, plan=False, lengths=3),
        # the package's headline step (workload 2): the plan, 32 layers on their own caches, accept, compaction
        dict(name="step_b16", kind="step", B=16, H_q=32, H_kv=8, D=128, dtype="bf16", layout="head", ctx="uniform",
             ctx_lo=1024, ctx_hi=4096, spec_lo=1, spec_hi=8, layers=32, plan=True, V=128256, lengths=4),
        # a loaded server (workload 3): one layer of a batch where many requests have no drafts (plain decode rows)
        dict(name="attn_b128", kind="attn", B=128, H_q=32, H_kv=8, D=128, dtype="bf16", layout="head", ctx="lognormal",
             ctx_lo=1, ctx_hi=8192, spec_lo=0, spec_hi=7, layers=1, plan=False, lengths=5),
        # wide query groups and long suffixes (workload 4 in one shot): up to 88 query rows per KV head
        dict(name="attn_wide_b256", kind="attn", B=256, H_q=64, H_kv=8, D=128, dtype="bf16", layout="head",
             ctx="lognormal", ctx_lo=16, ctx_hi=16384, spec_lo=1, spec_hi=10, layers=4, plan=True, lengths=6),
        # 8-bit caches in the token-major layout: quantising append, then attention
        dict(name="layer_kv8_b64", kind="layer", B=64, H_q=32, H_kv=8, D=128, dtype="kv8", layout="token",
             ctx="uniform", ctx_lo=512, ctx_hi=8192, spec_lo=1, spec_hi=8, layers=1, plan=False, lengths=7),
        # chunked verification at the largest batch (workload 5): frontiers of two drafts, accept per chunk
        dict(name="chunked_b512", kind="chunked", B=512, H_q=32, H_kv=8, D=128, dtype="bf16", layout="head",
             ctx="uniform", ctx_lo=512, ctx_hi=8192, spec_lo=2, spec_hi=8, layers=2, plan=True, V=152064, lengths=8),
        # sampling from logits, largest batch: softmax statistics of every tested row inside the call
        dict(name="accept_logits_b512", kind="accept", mode="logits", dtype="f32", B=512, V=152064, spec_lo=2,
             spec_hi=8, temperature=1.0, lengths=9),
        # the same from the bf16 logits a model's head produces, at a small batch (latency counts)
        dict(name="accept_logits_bf16_b16", kind="accept", mode="logits", dtype="bf16", B=16, V=128256, spec_lo=1,
             spec_hi=8, temperature=0.7, lengths=10),
        # temperature 0: arg-max acceptance, then the surviving rows are packed
        dict(name="greedy_b64", kind="accept", mode="greedy", dtype="f32", B=64, V=128256, spec_lo=1, spec_hi=8,
             temperature=1.0, lengths=11),
        # early exit inside the model: rank check on intermediate scores, prune the hidden states, restore them later
        dict(name="early_exit_b256", kind="early", dtype="bf16", B=256, V=128256, hidden=4096, spec_lo=1, spec_hi=10,
             lengths=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "attn_f32", "attn_d64", "step", "attn", "wide", "kv8", "chunked", "logits",
                       "logits_bf16", "probs", "greedy", "early"])
    lengths = rng.randrange(1 << 30)
    spec_lo = rng.randint(0, 3)
    spec = dict(spec_lo=spec_lo, spec_hi=spec_lo + rng.randint(0, 7), lengths=lengths)
    heads = rng.choice([(32, 8), (8, 2), (28, 4), (16, 16), (64, 8), (24, 8)])
    layout = rng.choice(["head", "token"])
    ctx_lo = _log_int(rng, 1, 1024)
    ctx = dict(ctx=rng.choice(["uniform", "lognormal"]), ctx_lo=ctx_lo, ctx_hi=max(ctx_lo, _log_int(rng, 256, 8192)))
    vocab = rng.choice([128256, 152064, 32000, rng.randint(20000, 160000)])
    base = dict(H_q=heads[0], H_kv=heads[1], D=128, dtype="bf16", layout=layout, layers=1, plan=False, **ctx, **spec)
    if kind == "layer":
        return dict(base, kind="layer", B=rng.randint(1, 8))
    if kind == "attn_f32":
        return dict(base, kind="attn", B=rng.randint(1, 8), dtype="f32", D=64, ctx_lo=rng.randint(1, 64),
                    ctx_hi=rng.randint(64, 512))
    if kind == "attn_d64":
        return dict(base, kind="attn", B=_log_int(rng, 1, 64), D=64)
    if kind == "step":
        return dict(base, kind="step", B=_log_int(rng, 4, 32), layers=rng.choice([16, 32]), plan=True, layout="head",
                    V=vocab, ctx_hi=max(ctx_lo, rng.randint(256, 4096)))
    if kind == "attn":
        return dict(base, kind="attn", B=_log_int(rng, 2, 192), layers=rng.choice([1, 2, 4]), plan=rng.random() < 0.5)
    if kind == "wide":
        return dict(base, kind="attn", B=_log_int(rng, 8, 256), H_q=64, H_kv=8, layers=2, plan=True,
                    spec_hi=spec_lo + rng.randint(5, 10))
    if kind == "kv8":
        return dict(base, kind="layer", B=_log_int(rng, 4, 96), dtype="kv8")
    if kind == "chunked":
        return dict(base, kind="chunked", B=_log_int(rng, 16, 256), H_q=32, H_kv=8, layers=2, plan=True, layout="head",
                    V=vocab, spec_lo=spec_lo + 1, spec_hi=spec_lo + rng.randint(3, 7))
    if kind == "early":
        return dict(kind="early", dtype=rng.choice(["bf16", "f32"]), B=_log_int(rng, 4, 256), V=vocab,
                    hidden=rng.choice([2048, 4096, 5120]), **spec)
    mode = {"logits_bf16": "logits"}.get(kind, kind)
    dtype = "bf16" if kind == "logits_bf16" else "f32"
    return dict(kind="accept", mode=mode, dtype=dtype, B=_log_int(rng, 4, 384), V=vocab,
                temperature=rng.choice([1.0, 0.7, 0.3]) if mode == "logits" else 1.0, **spec)


# ---------------------------------------------------------------------------------------------------------------
# lengths and offsets: a function of the case alone, so that its work is known without its data
# ---------------------------------------------------------------------------------------------------------------
def _lengths(case):
    rng = np.random.Generator(np.random.PCG64(case["lengths"]))
    B = case["B"]
    spec = rng.integers(case["spec_lo"], case["spec_hi"] + 1, size=B).astype(np.int32)
    if case.get("ctx") == "lognormal":
        ctx = np.clip(np.floor(rng.lognormal(math.log(2048), 1.0, size=B)), case["ctx_lo"], case["ctx_hi"])
        if case["spec_lo"] == 0:  # load-adaptive lengths: most requests draft little or nothing
            w = 0.7 ** np.arange(case["spec_hi"] + 1)
            spec = rng.choice(case["spec_hi"] + 1, size=B, p=w / w.sum()).astype(np.int32)
    else:
        ctx = rng.integers(case.get("ctx_lo", 1), case.get("ctx_hi", 1) + 1, size=B)
    return ctx.astype(np.int32), spec


def _offsets(lens):
    cu = np.zeros(len(lens) + 1, np.int32)
    np.cumsum(lens, out=cu[1:])
    return cu


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _normal(gen, shape, dtype, sigma=1.0):
    """N(0, sigma^2) values in `dtype`, drawn on the device in slabs."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    for a in range(0, flat.numel(), 1 << 28):
        n = min(1 << 28, flat.numel() - a)
        flat[a:a + n] = (torch.randn(n, generator=gen, device="cuda", dtype=torch.float32) * sigma).to(dtype)
    return out


def _paged(case, rng, gen):
    """Page tables over a permuted pool and one pair of caches per layer."""
    ctx, spec = _lengths(case)
    pages = (ctx + spec + 1 + PAGE - 1) // PAGE
    n_pages, max_pages = int(pages.sum()) + 3, int(pages.max())
    perm = rng.permutation(n_pages).astype(np.int32)
    bt = np.full((case["B"], max_pages), -1, np.int32)
    at = 0
    for i, n in enumerate(pages):
        bt[i, :n] = perm[at:at + n]
        at += int(n)
    H, D = case["H_kv"], case["D"]
    shape = (n_pages, H, PAGE, D) if case["layout"] == "head" else (n_pages, PAGE, H, D)
    caches = []
    for _ in range(2 * case["layers"]):
        if case["dtype"] == "kv8":
            caches.append(_codes(gen, shape))
        else:
            caches.append(_normal(gen, shape, DTYPES[case["dtype"]]))
    cu_q = _offsets(spec + 1)
    act = torch.bfloat16 if case["dtype"] == "kv8" else DTYPES[case["dtype"]]
    N = int(cu_q[-1])
    s = dict(case=case, ctx=_dev(ctx), spec=_dev(spec), cu_q=_dev(cu_q), cu_d=_dev(_offsets(spec)), bt=_dev(bt),
             k=caches[0::2], v=caches[1::2], q=_normal(gen, (N, case["H_q"], D), act), N=N, S_max=int(spec.max()),
             scale=1.0 / math.sqrt(D), kv_layout=binding.KV_HEAD_MAJOR if case["layout"] == "head" else binding.KV_TOKEN_MAJOR)
    s["out"] = [torch.zeros_like(s["q"]) for _ in range(case["layers"])]
    s["lse"] = torch.zeros((N, case["H_q"]), dtype=torch.float32, device="cuda")
    need = fsr.attn_workspace_bytes(B=case["B"], N_cap=N, H_q=case["H_q"], H_kv=H, D=D, P=PAGE, max_pages=max_pages,
                                    n_pages=n_pages, dtype=act, out_dtype=act, max_q_len=s["S_max"] + 1)
    s["ws"] = torch.empty(max(256, need), dtype=torch.uint8, device="cuda")
    return s


def _codes(gen, shape):
    """E4M3 bytes of N(0, 1) keys or values stored with KV8_SCALE."""
    out = torch.empty(shape, dtype=torch.uint8, device="cuda")
    flat = out.view(-1)
    for a in range(0, flat.numel(), 1 << 28):
        n = min(1 << 28, flat.numel() - a)
        x = torch.randn(n, generator=gen, device="cuda", dtype=torch.float32) / KV8_SCALE
        flat[a:a + n] = x.clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    return out


def _rows(case, gen, probs):
    """Target and draft rows (logits N(0, 2^2) and target + N(0, 0.5^2), or their softmax), draft tokens, uniforms."""
    _, spec = _lengths(case)
    cu_q, cu_d, V = _offsets(spec + 1), _offsets(spec), case["V"]
    N, N_d = int(cu_q[-1]), int(cu_d[-1])
    dtype = DTYPES["f32" if case["kind"] != "accept" else case["dtype"]]
    owner = np.repeat(np.arange(len(spec)), spec)
    pair = _dev((cu_q[owner] + np.arange(N_d) - cu_d[owner]).astype(np.int64))  # target row that verifies the draft
    t = _normal(gen, (N, V), dtype, 2.0)
    d = torch.empty((N_d, V), dtype=dtype, device="cuda")
    tok = torch.empty(N_d, dtype=torch.int32, device="cuda")
    step = max(1, (1 << 27) // V)
    for a in range(0, N_d, step):
        x = t[pair[a:a + step]].float()
        z = (x + torch.randn(x.shape, generator=gen, device="cuda") * 0.5).to(dtype)
        noise = torch.rand(x.shape, generator=gen, device="cuda").clamp_(1e-12, 1 - 6e-8)
        z_T = z.float() / case.get("temperature", 1.0)
        if case.get("mode") != "greedy":  # a sample of softmax(z / T); at temperature 0 the drafter's own best token
            z_T = z_T - torch.log(-torch.log(noise))
        tok[a:a + step] = z_T.argmax(1).to(torch.int32)
        d[a:a + step] = z
    if probs:
        for rows in (t, d):
            for a in range(0, rows.shape[0], step):
                rows[a:a + step] = torch.softmax(rows[a:a + step].double(), dim=1).to(dtype)
    return dict(t=t, d=d, tok=tok, u_a=torch.rand(N_d, generator=gen, device="cuda"),
                u_s=torch.rand(case["B"], generator=gen, device="cuda"), cu_t=_dev(cu_q), cu_d=_dev(cu_d), N=N, N_d=N_d,
                S_max=int(spec.max()))


def _maps(B, N):
    i32 = dict(dtype=torch.int32, device="cuda")
    return dict(new_cu_q=torch.empty(B + 1, **i32), new_q_lens=torch.empty(B, **i32), src_row=torch.empty(N, **i32),
                dst_row=torch.empty(N, **i32), n_active=torch.empty(1, **i32), active_ids=torch.empty(B, **i32))


def _accept_ws(B, V, S_max, mode, temperature=1.0):
    need = fsr.accept_workspace_bytes(B=B, V=V, S_max=S_max, mode=mode, temperature=temperature)
    return torch.empty(max(256, need), dtype=torch.uint8, device="cuda")


MODES = {"probs": binding.PROBS, "logits": binding.LOGITS, "greedy": binding.GREEDY}


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rng = np.random.Generator(np.random.PCG64(seed))
    kind = case["kind"]
    if kind == "accept":
        s = _rows(case, gen, probs=case["mode"] != "logits")
        s.update(case=case, mode=MODES[case["mode"]],
                 ws=_accept_ws(case["B"], case["V"], s["S_max"], MODES[case["mode"]], case["temperature"]))
        if case["mode"] == "greedy":  # the step's hidden states, packed behind the accept
            s.update(hidden=_normal(gen, (s["N"], 4096), torch.bfloat16), maps=_maps(case["B"], s["N"]))
            s["packed"] = torch.zeros_like(s["hidden"])
        return s
    if kind == "early":
        _, spec = _lengths(case)
        cu_q, cu_d = _offsets(spec + 1), _offsets(spec)
        N, N_d, V = int(cu_q[-1]), int(cu_d[-1]), case["V"]
        logits = _normal(gen, (N, V), DTYPES[case["dtype"]], 2.0)
        owner = np.repeat(np.arange(len(spec)), spec)
        rows = _dev((cu_q[owner] + np.arange(N_d) - cu_d[owner]).astype(np.int64))
        # most drafts are among the best tokens of their row, some are not
        tok = torch.randint(0, V, (N_d,), generator=gen, device="cuda", dtype=torch.int32)
        step = max(1, (1 << 27) // V)
        for a in range(0, N_d, step):
            best = torch.topk(logits[rows[a:a + step]].float(), 8, dim=1).indices
            pick = torch.randint(0, 10, (best.shape[0],), generator=gen, device="cuda")
            chosen = best.gather(1, pick.clamp(max=7)[:, None])[:, 0].to(torch.int32)
            tok[a:a + step] = torch.where(pick < 8, chosen, tok[a:a + step])
        hidden = _normal(gen, (N, case["hidden"]), torch.bfloat16)
        return dict(case=case, logits=logits, tok=tok, cu_q=_dev(cu_q), cu_d=_dev(cu_d), hidden=hidden, N=N,
                    maps=_maps(case["B"], N), packed=torch.zeros_like(hidden), restored=torch.zeros_like(hidden),
                    rank=torch.zeros(N_d, dtype=torch.int32, device="cuda"))
    s = _paged(case, rng, gen)
    if kind == "layer":
        act = s["q"].dtype
        s["k_new"] = _normal(gen, (s["N"], case["H_kv"], case["D"]), act)
        s["v_new"] = _normal(gen, (s["N"], case["H_kv"], case["D"]), act)
        s["sc"] = torch.full((case["H_kv"],), KV8_SCALE, dtype=torch.float32, device="cuda")
    if kind in ("step", "chunked"):
        s["rows"] = _rows(case, gen, probs=True)
    if kind == "step":
        s["ws_acc"] = _accept_ws(case["B"], case["V"], s["S_max"], binding.PROBS)
        s["maps"] = _maps(case["B"], s["N"])
        s["packed"] = torch.zeros_like(s["out"][0])
    if case["plan"] and kind != "chunked":
        s["plan"] = fsr.attn_plan(s["q"], s["k"][0], s["bt"], s["ctx"], s["cu_q"], scale=s["scale"],
                                  max_q_len=s["S_max"] + 1, kv_layout=s["kv_layout"])
    if kind == "chunked":
        _, spec = _lengths(case)
        r = s["rows"]
        chunks = [_dev(np.clip(spec - a, 0, 2).astype(np.int32)) for a in range(0, max(1, int(spec.max())), 2)]
        s["verifier"] = ChunkedVerifier(
            q=s["q"], k_caches=s["k"], v_caches=s["v"], block_tables=s["bt"], ctx_lens=s["ctx"], spec_lens=s["spec"],
            cu_q=s["cu_q"], cu_d=s["cu_d"], p_target=r["t"], p_draft=r["d"], draft_tokens=r["tok"], u_accept=r["u_a"],
            u_sample=r["u_s"], chunks=chunks, scale=s["scale"], out=s["out"][0], S_total_max=s["S_max"],
            chunk_S_max=min(2, s["S_max"]))
    return s


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------
def _attention(s):
    case = s["case"]
    plan = None
    if case["plan"]:  # once per step, read by every layer
        plan = fsr.attn_plan(s["q"], s["k"][0], s["bt"], s["ctx"], s["cu_q"], scale=s["scale"], max_q_len=s["S_max"] + 1,
                             kv_layout=s["kv_layout"], plan=s["plan"])
    for l in range(case["layers"]):
        fsr.verify_attention(s["q"], s["k"][l], s["v"][l], s["bt"], s["ctx"], s["spec"], s["cu_q"], scale=s["scale"],
                             out=s["out"][l], lse=s["lse"] if l == 0 else None, workspace=s["ws"],
                             max_q_len=s["S_max"] + 1, kv_layout=s["kv_layout"], plan=plan)
    return dict(out=s["out"], lse=s["lse"])


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "attn":
        return _attention(s)
    if kind == "layer":
        if case["dtype"] == "kv8":
            fsr.kv_append_kv8(s["k_new"], s["v_new"], s["k"][0], s["v"][0], s["sc"], s["sc"], s["bt"], s["ctx"], s["cu_q"],
                              kv_layout=s["kv_layout"])
            fsr.verify_attention_kv8(s["q"], s["k"][0], s["v"][0], s["sc"], s["sc"], s["bt"], s["ctx"], s["cu_q"],
                                     scale=s["scale"], out=s["out"][0], lse=s["lse"], workspace=s["ws"],
                                     max_q_len=s["S_max"] + 1, kv_layout=s["kv_layout"])
            return dict(out=s["out"], lse=s["lse"], k=s["k"][0], v=s["v"][0])
        fsr.kv_append(s["k_new"], s["v_new"], s["k"][0], s["v"][0], s["bt"], s["ctx"], s["cu_q"], kv_layout=s["kv_layout"])
        return dict(_attention(s), k=s["k"][0], v=s["v"][0])
    if kind == "step":
        got, r = _attention(s), s["rows"]
        acc, n, em = fsr.spec_accept(r["t"], r["d"], r["tok"], r["u_a"], r["u_s"], s["cu_q"], s["cu_d"], S_max=s["S_max"],
                                     workspace=s["ws_acc"])
        kept = fsr.survivor_compact(acc, s["cu_q"], s["N"], payload=s["out"][-1], payload_out=s["packed"], out=s["maps"])
        return dict(got, accepted=acc, n=n, emitted=em, **kept)
    if kind == "chunked":
        return s["verifier"].run()
    if kind == "accept":
        draft = (None, s["tok"], None, None) if case["mode"] == "greedy" else (s["d"], s["tok"], s["u_a"], s["u_s"])
        acc, n, em = fsr.spec_accept(s["t"], *draft, s["cu_t"], s["cu_d"], S_max=s["S_max"], mode=s["mode"],
                                     temperature=case["temperature"], workspace=s["ws"])
        got = dict(accepted=acc, n=n, emitted=em)
        if case["mode"] == "greedy":
            got.update(fsr.survivor_compact(acc, s["cu_t"], s["N"], payload=s["hidden"], payload_out=s["packed"],
                                            out=s["maps"]))
        return got
    rank, keep = fsr.topk_rank_check(s["logits"], s["tok"], s["cu_q"], s["cu_d"], K=RANK_K, rank=s["rank"])
    kept = fsr.prune_compact(keep, s["cu_q"], payload=s["hidden"], payload_out=s["packed"], out=s["maps"])
    restored, has = fsr.prune_restore(kept["payload"], kept["dst_row"], restored=s["restored"])
    return dict(kept, rank=rank, keep=keep, restored=restored, has=has)


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------
def _attention_work(case):
    ctx, spec = (x.astype(np.int64) for x in _lengths(case))
    e_kv = {"bf16": 2, "f32": 4, "kv8": 1}[case["dtype"]]
    e = 4 if case["dtype"] == "f32" else 2
    tok, rows = int((ctx + spec + 1).sum()), int((spec + 1).sum())
    keys = int(((spec + 1) * ctx + (spec + 1) * (spec + 2) // 2).sum())
    per_layer = 2 * tok * case["H_kv"] * case["D"] * e_kv + 2 * rows * case["H_q"] * case["D"] * e
    table = 4 * int(((ctx + spec + PAGE) // PAGE).sum())
    return case["layers"] * per_layer + table, case["layers"] * 4 * case["H_q"] * case["D"] * keys, rows


def _tested_rows(spec, alpha=ALPHA):
    """Expected drafts that are tested and requests that are accepted to the end."""
    spec = spec.astype(np.float64)
    return float(((1 - alpha ** spec) / (1 - alpha)).sum()), float((alpha ** spec).sum())


def work(case):
    kind = case["kind"]
    if kind in ("attn", "layer"):
        nbytes, flops, rows = _attention_work(case)
        if kind == "layer":  # the call's own rows in, and into the caches
            e_kv = {"bf16": 2, "kv8": 1}[case["dtype"]]
            nbytes += 2 * rows * case["H_kv"] * case["D"] * (2 + e_kv)
        return {"bytes": nbytes, "flops": flops}
    _, spec = _lengths(case)
    N, N_d, B = int((spec + 1).sum()), int(spec.sum()), case["B"]
    if kind == "early":
        e = 2 if case["dtype"] == "bf16" else 4
        # one score row per draft, about the first half of the hidden rows packed, all of them restored
        return {"bytes": N_d * case["V"] * e + 2 * (N // 2) * case["hidden"] * 2 + N * case["hidden"] * 2,
                "flops": N_d * case["V"]}
    V = case["V"]
    tested, through = _tested_rows(spec)
    if kind == "accept":
        e = 2 if case["dtype"] == "bf16" else 4
        if case["mode"] == "greedy":  # a request's rows up to its first mismatch (about one in two drafts is the arg-max)
            tested, through = _tested_rows(spec, 0.5)
            return {"bytes": (tested + through) * V * e + 2 * (tested + through) * 8192, "flops": (tested + through) * V}
        if case["mode"] == "logits":  # softmax of every row that decides, and of those sampled from
            return {"bytes": (2 * tested + through) * V * e, "flops": 4 * (2 * tested + through) * V}
        return {"bytes": (2 * (B - through) + through) * V * e, "flops": 2 * (2 * B - through) * V}
    nbytes, flops, _ = _attention_work(case)
    nbytes += (2 * (B - through) + through) * V * 4  # the row pair (or bonus row) each request samples from
    if kind == "step":
        nbytes += 2 * (tested + through) * case["H_q"] * case["D"] * 2
    # the chunked schedule reads a request's K/V again in every chunk it reaches: frontiers of two drafts
    if kind == "chunked":
        ctx, spec = (x.astype(np.float64) for x in _lengths(case))
        kv = 2 * (ctx + 2) * case["H_kv"] * case["D"] * 2 * case["layers"]
        for a in range(2, int(spec.max()), 2):
            nbytes += float((kv * (spec > a) * ALPHA ** a).sum())
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind in ("accept", "early"):
        return "exact"  # tokens, ranks, maps and copied rows: decisions in 64 bits, no rounding to differ in
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 4e-5}  # 2.5e-7 against 64 bits
    # bf16 results: one rounding of the output, 1.7e-3 against 64 bits; lse (fp32) is far inside it
    return {"rel": 7e-3, "max": 1.6e-2}


# ---------------------------------------------------------------------------------------------------------------
# 64-bit results
# ---------------------------------------------------------------------------------------------------------------
def _wide(x, kv8):
    return x.view(torch.float8_e4m3fn).double() * float(np.float32(KV8_SCALE)) if kv8 else x.double()


def _exact_attention(s, k, v, rows_of=None):
    """softmax(scale q K^T) V over the paged caches, and the log of the sums, in 64 bits."""
    case = s["case"]
    ctx, spec = _lengths(case)
    cu, kv8 = _offsets(spec + 1), case["dtype"] == "kv8"
    out = torch.zeros(s["q"].shape, dtype=torch.float64, device="cuda")
    lse = torch.zeros(s["q"].shape[:2], dtype=torch.float64, device="cuda")
    Hk, D, G = case["H_kv"], case["D"], case["H_q"] // case["H_kv"]
    for i in range(case["B"]):
        n, L = int(spec[i]) + 1, int(ctx[i] + spec[i] + 1)
        pages = s["bt"][i, :(L + PAGE - 1) // PAGE].long()
        kk, vv = (_wide(x[pages], kv8) for x in (k, v))
        if case["layout"] == "head":
            kk, vv = kk.transpose(1, 2), vv.transpose(1, 2)
        kk, vv = (x.reshape(-1, Hk, D)[:L].permute(1, 0, 2).contiguous() for x in (kk, vv))
        q = s["q"][cu[i]:cu[i + 1]].double().view(n, Hk, G, D).permute(1, 0, 2, 3).reshape(Hk, n * G, D)
        z = torch.matmul(q, kk.transpose(1, 2).contiguous()).view(Hk, n, G, L) * s["scale"]
        last = torch.arange(n, device="cuda")[:, None] + int(ctx[i])
        z = z.masked_fill((torch.arange(L, device="cuda")[None] > last)[None, :, None], float("-inf"))
        o = torch.matmul(torch.softmax(z, -1).view(Hk, n * G, L), vv).view(Hk, n, G, D)
        out[cu[i]:cu[i + 1]] = o.permute(1, 0, 2, 3).reshape(n, case["H_q"], D)
        lse[cu[i]:cu[i + 1]] = torch.logsumexp(z, -1).permute(1, 0, 2).reshape(n, case["H_q"])
    return out, lse


def _accepted(r, spec):
    """Leading accepted drafts of every request: u q(x) < p(x) in 64 bits."""
    cu_q, cu_d = _offsets(spec + 1), _offsets(spec)
    owner = np.repeat(np.arange(len(spec)), spec)
    pair = _dev((cu_q[owner] + np.arange(r["N_d"]) - cu_d[owner]).astype(np.int64))
    tok = r["tok"].long()
    p, q = r["t"][pair, tok].double(), r["d"][torch.arange(r["N_d"], device="cuda"), tok].double()
    ok = (r["u_a"].double() * q < p).cpu().numpy()
    got = np.zeros(len(spec), np.int64)
    for i in range(len(spec)):
        run_ = ok[cu_d[i]:cu_d[i + 1]]
        got[i] = len(run_) if run_.all() else int(np.argmin(run_))
    return got


def exact(case, seed):
    kind = case["kind"]
    if kind in ("accept", "early"):
        return None
    s = prepare(case, seed)
    ctx, spec = _lengths(case)
    if kind == "layer":  # the appended rows, as the caches store them
        cu = _offsets(spec + 1)
        for new, cache in ((s["k_new"], s["k"][0]), (s["v_new"], s["v"][0])):
            stored = new if case["dtype"] != "kv8" else (new.float() / s["sc"][None, :, None]).clamp(-448, 448).to(
                torch.float8_e4m3fn).view(torch.uint8)
            for i in range(case["B"]):
                for j in range(int(spec[i]) + 1):
                    t = int(ctx[i]) + j
                    page = int(s["bt"][i, t // PAGE])
                    if case["layout"] == "head":
                        cache[page, :, t % PAGE] = stored[int(cu[i]) + j]
                    else:
                        cache[page, t % PAGE] = stored[int(cu[i]) + j]
    layers = [case["layers"] - 1] if kind == "chunked" else range(case["layers"])
    got = [_exact_attention(s, s["k"][l], s["v"][l]) for l in layers]
    if kind == "chunked":
        # a request's rows are computed up to the chunk of its first rejection; the others keep the zeros they had
        out, n = got[0][0], _accepted(s["rows"], spec)
        cu = _offsets(spec + 1)
        for i in range(case["B"]):
            done = 2 * (int(n[i]) // 2) + 2
            if n[i] < spec[i] and done < spec[i]:  # (the chunk with the last draft carries the bonus row too)
                out[cu[i] + done:cu[i + 1]] = 0
        return dict(accepted_len=None, n_emitted=None, emitted=None, out=out)
    res = dict(out=[o for o, _ in got], lse=got[0][1])
    if kind == "layer":
        res.update(k=None, v=None)
    if kind == "step":
        n = _accepted(s["rows"], spec)
        cu = _offsets(spec + 1)
        keep = np.concatenate([np.arange(cu[i], cu[i] + n[i] + 1) for i in range(case["B"])])
        packed = torch.zeros_like(got[-1][0])
        packed[:len(keep)] = got[-1][0][_dev(keep.astype(np.int64))]
        res.update(accepted=None, n=None, emitted=None, new_cu_q=None, new_q_lens=None, src_row=None, dst_row=None,
                   n_active=None, active_ids=None, payload=packed)
    return res
