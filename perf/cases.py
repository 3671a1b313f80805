"""The calls whose speed is watched: what a rollout and training loop asks of this library.

Every case is one pass through the public entry points of paper_2602_09578_amd.binding over
seeded synthetic inputs.  `listed()` names the fixed ones, `draw()` gives more of the same
ranges: batches from one prompt to a few thousand sequences, contexts from a few tokens to
tens of thousands, the head counts of the repository's workloads and tests, vocabularies whose
rows start aligned and unaligned, bf16 and float32 outputs.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2602_09578_amd import binding as B
from paper_2602_09578_amd import inputs as I

D, PAGE = 128, 16
LENS_SEED = 2048   # lengths belong to the case (its work is fixed); values and page placement to the seed


# ---- the cases ---------------------------------------------------------------------------------
def listed():
    return [
        # One decode step of a handful of samples: two agents, two prompts each, four samples per
        # prompt, short contexts.  Four launches and the plan's chain of loads are the whole cost.
        dict(name="decode_few", op="decode", Hq=8, Hkv=2, out="bf16",
             agents="2x4 const:256 uniform:1:128; 2x4 const:256 uniform:1:128"),
        # The ordinary decode step: 2048 samples of 256 prompts, four agents whose responses have
        # medians of 256 to 2048 tokens with a long tail.  Bound by the KV bytes.
        dict(name="decode_batch", op="decode", Hq=28, Hkv=4, out="bf16",
             agents="; ".join(f"64x8 uniform:512:2048 lognormal:{m}:0.8:8192" for m in (256, 512, 1024, 2048))),
        # The first steps after a long prompt was expanded into 32 samples: nearly all of the work
        # is the shared prefix, a dense product of 224 query rows per KV head.
        dict(name="decode_group_sampling", op="decode", Hq=28, Hkv=4, out="bf16", agents="64x32 const:4096 uniform:1:64"),
        # Long contexts on a larger model's heads: 8192-token prompts, 8k to 24k generated tokens.
        dict(name="decode_long", op="decode", Hq=64, Hkv=8, out="f32",
             agents="; ".join(["16x4 const:8192 uniform:8192:24576"] * 4)),
        # A whole rollout step at the paper's parallelism (4 prompts x 16 samples): the new token is
        # appended to the cache, attention runs over it, and the next token is drawn from its logits
        # together with its log-probability.
        dict(name="rollout_step", op="step", Hq=64, Hkv=8, out="bf16",
             agents="4x16 uniform:512:2048 lognormal:1024:0.8:8192", vocab=152064, sigma=3.0, T=1.0, top_p=0.95),
        # Log-probabilities of one token per row: the decode batch, and an odd vocabulary (rows start
        # at any alignment) in an evaluation at another temperature.
        dict(name="logprobs_batch", op="logprobs", rows=2048, vocab=152064, sigma=3.0, T=1.0),
        dict(name="logprobs_odd_vocab", op="logprobs", rows=333, vocab=20481, sigma=3.0, T=0.7),
        # Drawing the next token: from the whole distribution (a small batch), from the nucleus (the
        # full batch).
        dict(name="sample_small_batch", op="sample", rows=256, vocab=152064, sigma=3.0, T=1.0),
        dict(name="sample_nucleus", op="top_p", rows=2048, vocab=152064, sigma=3.0, T=1.0, top_p=0.9),
        # Prompt attention of a whole batch of prompts, from position 0.
        dict(name="prefill_prompts", op="prefill", Hq=28, Hkv=4, out="bf16", prompts=256, chunk="uniform:512:2048",
             context="const:0", write=False),
        # Chunked prefill beside decoding: a few prompts each bring a piece of up to 512 tokens behind
        # context that is already cached; keys and values are scattered into the pages first.
        dict(name="prefill_chunks", op="prefill", Hq=64, Hkv=8, out="bf16", prompts=6, chunk="uniform:33:512",
             context="uniform:0:8192", write=True),
        # Weight synchronisation: a model's parameter list gathered into one buffer and scattered back.
        dict(name="weight_sync", op="pack", Hq=8, Hkv=2, vocab=4096),
    ]


HEADS = [(8, 2), (28, 4), (28, 4), (64, 8), (64, 8), (32, 8), (16, 1), (4, 4)]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def _draw_decode(rng):
    Hq, Hkv = rng.choice(HEADS)
    agents = []
    budget = 8e9 / (2 * Hkv * D * 2)   # tokens
    for _ in range(rng.randint(1, 4)):
        G = _log_int(rng, 1, 32)
        prompts = _log_int(rng, 1, 64)
        hi = _log_int(rng, 16, 8192)
        plen = rng.choice([f"const:{hi}", f"uniform:{max(1, hi // 4)}:{hi}"])
        top = _log_int(rng, 8, 16384)
        if rng.random() < 0.5:
            glen, mean = f"uniform:{max(1, top // 8)}:{top}", top * 0.6
        else:
            glen, mean = f"lognormal:{max(1, top // 4)}:0.8:{top}", top * 0.35
        cost = prompts * (hi + G * mean)
        if cost > budget / 4:
            prompts = max(1, int(prompts * budget / 4 / cost))
        agents.append(f"{prompts}x{G} {plen} {glen}")
    return dict(Hq=Hq, Hkv=Hkv, out=rng.choice(["bf16", "bf16", "f32"]), agents="; ".join(agents))


def draw(rng):
    op = rng.choice(["decode", "decode", "decode", "logprobs", "sample", "top_p", "prefill", "prefill", "step", "pack"])
    if op == "decode":
        return dict(op=op, **_draw_decode(rng))
    vocab = rng.choice([4096, 4099, 20481, 32000, 32003, 65536, 100003, 128001, 152064, 152064, 152064 + 8 * rng.randint(1, 999)])
    if op == "step":
        c = dict(op=op, **_draw_decode(rng))
        c.update(vocab=vocab, sigma=rng.choice([2.0, 3.0]), T=rng.choice([0.7, 1.0]), top_p=rng.choice([0.9, 0.95]))
        first, *rest = c["agents"].split("; ")
        c["agents"] = first   # one agent: at most 64 x 32 rows of logits
        return c
    if op in ("logprobs", "sample", "top_p"):
        rows = _log_int(rng, 1, min(4096, 311427072 // vocab))
        c = dict(op=op, rows=rows, vocab=vocab, sigma=rng.choice([2.0, 3.0]), T=rng.choice([0.7, 1.0, 1.3]))
        if op == "top_p":
            c["top_p"] = rng.choice([0.8, 0.9, 0.95])
        return c
    if op == "prefill":
        Hq, Hkv = rng.choice(HEADS)
        hi, prompts = _log_int(rng, 16, 4096), _log_int(rng, 1, 64)
        ctx = rng.choice([0, 0, _log_int(rng, 16, 8192)])
        cap = 1.0e12 / (4 * D * Hq)   # (query, key) pairs
        prompts = max(1, min(prompts, int(cap / (hi * (hi / 2 + ctx / 2) + 1))))
        return dict(op=op, Hq=Hq, Hkv=Hkv, out=rng.choice(["bf16", "bf16", "f32"]), prompts=prompts,
                    chunk=f"uniform:{max(1, hi // 4)}:{hi}", context=f"uniform:0:{ctx}" if ctx else "const:0",
                    write=rng.random() < 0.5)
    Hq, Hkv = rng.choice([(4, 4), (8, 2), (8, 2)])
    return dict(op="pack", Hq=Hq, Hkv=Hkv, vocab=vocab)


# ---- lengths -----------------------------------------------------------------------------------
def _dist(text):
    kind, *v = text.split(":")
    v = [float(x) for x in v]
    return {"const": I.const, "uniform": I.uniform, "lognormal": I.lognormal}[kind](*v)


def _lengths(case):
    agents = []
    for part in case["agents"].split("; "):
        shape, plen, glen = part.split()
        prompts, G = shape.split("x")
        agents.append(I.Agent(int(prompts), int(G), _dist(plen), _dist(glen)))
    w = I.Workload("case", case["Hq"], case["Hkv"], tuple(agents), seed=LENS_SEED)
    return w, I.draw_lengths(w, np.random.default_rng(LENS_SEED))


def _prefill_lengths(case):
    rng = np.random.default_rng(LENS_SEED)
    n = case["prompts"]
    return _dist(case["chunk"]).draw(rng, n), _dist(case["context"]).draw(rng, n)


def _out_dtype(case):
    return B.MARL_OUT_F32 if case["out"] == "f32" else B.MARL_OUT_BF16


# ---- inputs ------------------------------------------------------------------------------------
def _logits(rows, vocab, sigma, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return I.randn_bf16((rows, vocab), sigma, gen, "cuda"), gen


def _draw_uniforms(logits, T, top_p, gen):
    """(uniforms, tokens, log-probabilities).  Tokens are drawn from the (nucleus) distribution and each
    uniform number is the middle of its token's interval, so that which token is drawn does not hang on
    the last bit of a float sum and outputs can be compared exactly.  In a nucleus the tokens within a
    factor 2.5 of its smallest probability are left out for the same reason (one token more or less at
    the threshold moves every interval by up to that probability)."""
    rows, vocab = logits.shape
    u = torch.empty(rows, dtype=torch.float32, device="cuda")
    tok = torch.empty(rows, dtype=torch.int64, device="cuda")
    lp = torch.empty(rows, dtype=torch.float64, device="cuda")
    step = max(1, (1 << 26) // vocab)
    for a in range(0, rows, step):
        p = torch.softmax(logits[a:a + step].double() / T, dim=1)
        kept, pool = p, p
        if top_p < 1.0:
            srt, order = torch.sort(p, dim=1, descending=True, stable=True)
            last = (torch.cumsum(srt, 1) < top_p).sum(1, keepdim=True).clamp(max=vocab - 1)
            inside = torch.arange(vocab, device="cuda")[None, :] <= last
            kept = p * torch.zeros_like(inside).scatter_(1, order, inside)
            pool = torch.where(kept >= 2.5 * srt.gather(1, last), kept, torch.zeros_like(kept))
            pool = torch.where(pool.sum(1, keepdim=True) > 0, pool, kept)
        pool_cdf = torch.cumsum(pool, 1)
        r = torch.rand(p.shape[0], 1, generator=gen, device="cuda", dtype=torch.float64) * pool_cdf[:, -1:]
        t = torch.searchsorted(pool_cdf, r, right=True).clamp(max=vocab - 1)
        cdf = torch.cumsum(kept, 1)
        mid = (cdf.gather(1, t) - 0.5 * kept.gather(1, t)) / cdf[:, -1:]
        u[a:a + step] = mid[:, 0].float().clamp(max=1.0 - 2.0 ** -24)
        tok[a:a + step] = t[:, 0]
        lp[a:a + step] = torch.log(p.gather(1, t))[:, 0]
    return u, tok, lp


def _model_tensors(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [I.randn_bf16((n,), 0.02, gen, "cuda") for n in I.model_param_sizes(case["Hq"], case["Hkv"], case["vocab"])]


def _attn_state(case, seed, poison):
    w, lens = _lengths(case)
    inp = I.build_attn_inputs(w, device="cuda", seed=seed, poison=poison, lengths=lens)
    return dict(case=case, inp=inp, call=B.prepare_attn(inp, _out_dtype(case)))


def prepare(case, seed):
    op = case["op"]
    if op == "decode":
        return _attn_state(case, seed, True)
    if op == "step":
        s = _attn_state(case, seed, False)   # (the whole cache is returned: no NaN in it)
        inp, n = s["inp"], s["inp"].num_seqs
        s["lens_now"] = inp.suffix_lens - 1          # the scheduler's lengths before this step's token
        gen = torch.Generator(device="cuda").manual_seed(seed + 1)
        s["k_new"] = I.randn_bf16((n, inp.Hkv, D), 1.0, gen, "cuda")
        s["v_new"] = I.randn_bf16((n, inp.Hkv, D), 1.0, gen, "cuda")
        s.update(_sampling_state(n, case, seed + 2))
        return s
    if op == "logprobs":
        logits, gen = _logits(case["rows"], case["vocab"], case["sigma"], seed)
        tokens = torch.randint(0, case["vocab"], (case["rows"],), generator=gen, device="cuda", dtype=torch.int32)
        need = B.marl_logprobs_workspace_bytes(case["rows"], case["vocab"])
        return dict(case=case, logits=logits, tokens=tokens, ws=B.alloc_workspace(need, "cuda") if need else None,
                    out=torch.empty(case["rows"], dtype=torch.float32, device="cuda"))
    if op in ("sample", "top_p"):
        return dict(case=case, **_sampling_state(case["rows"], case, seed))
    if op == "prefill":
        chunk, ctx = _prefill_lengths(case)
        inp = I.build_prefill_inputs(case["Hq"], case["Hkv"], chunk, ctx, device="cuda", seed=seed, poison=not case["write"])
        shape, ws, out = B.prepare_prefill(inp, _out_dtype(case))
        return dict(case=case, inp=inp, shape=shape, ws=ws, out=out)
    tensors = _model_tensors(case, seed)
    table = B.PackTable(tensors)
    flat = torch.zeros(sum(t.numel() for t in tensors), dtype=torch.bfloat16, device="cuda")   # the receiver's parameters
    return dict(case=case, tensors=tensors, table=table, flat=flat,
                back_table=B.PackTable(list(flat.split([t.numel() for t in tensors]))),
                packed=torch.zeros(table.packed_bytes, dtype=torch.uint8, device="cuda"))


def _sampling_state(rows, case, seed):
    logits, gen = _logits(rows, case["vocab"], case["sigma"], seed)
    u, _, _ = _draw_uniforms(logits, case["T"], case.get("top_p", 1.0), gen)
    s = dict(logits=logits, u=u, tok=torch.empty(rows, dtype=torch.int32, device="cuda"),
             lp=torch.empty(rows, dtype=torch.float32, device="cuda"))
    if case["op"] == "sample":
        s["sample_ws"] = B.alloc_workspace(B.marl_sample_workspace_bytes(rows, case["vocab"]), "cuda")
    return s


# ---- one pass ----------------------------------------------------------------------------------
def run(s):
    case, op = s["case"], s["case"]["op"]
    if op == "decode":
        return B.run_attn(s["inp"], s["call"])
    if op == "step":
        inp, call = s["inp"], s["call"]
        inp.suffix_lens.copy_(s["lens_now"])
        B.marl_kv_append(call.shape, s["k_new"], s["v_new"], inp.k_pages, inp.v_pages, inp.suffix_block_table, inp.suffix_lens)
        out = B.run_attn(inp, call)
        B.marl_sample_tokens_top_p(s["logits"], s["u"], case["T"], case["top_p"], s["tok"], s["lp"])
        return dict(out=out, tokens=s["tok"], logprobs=s["lp"], lens=inp.suffix_lens, k=inp.k_pages, v=inp.v_pages)
    if op == "logprobs":
        return B.marl_token_logprobs(s["logits"], s["tokens"], case["T"], s["out"], s["ws"])
    if op == "sample":
        B.marl_sample_tokens(s["logits"], s["u"], case["T"], s["tok"], s["lp"], s["sample_ws"])
        return dict(tokens=s["tok"], logprobs=s["lp"])
    if op == "top_p":
        B.marl_sample_tokens_top_p(s["logits"], s["u"], case["T"], case["top_p"], s["tok"], s["lp"])
        return dict(tokens=s["tok"], logprobs=s["lp"])
    if op == "prefill":
        inp = s["inp"]
        if case["write"]:
            B.marl_kv_write_prompt(s["shape"], inp.k_new, inp.v_new, inp.k_pages, inp.v_pages,
                                   inp.prefix_block_table, inp.q_start, inp.q_pos0)
        out = B.run_prefill(inp, s["shape"], s["ws"], s["out"])
        return dict(out=out, k=inp.k_pages, v=inp.v_pages) if case["write"] else out
    B.marl_pack_tensors(s["table"], s["packed"])
    B.marl_unpack_tensors(s["back_table"], s["packed"])
    return dict(packed=s["packed"], parameters=s["flat"])


# ---- what a pass cannot do without -------------------------------------------------------------
def work(case):
    op = case["op"]
    logit_bytes = 0
    if op in ("logprobs", "sample", "top_p"):
        n = case["rows"] * case["vocab"]
        return dict(bytes=2 * n + 12 * case["rows"], flops=3 * n)
    if op == "pack":
        n = sum(I.model_param_sizes(case["Hq"], case["Hkv"], case["vocab"]))
        return dict(bytes=4 * 2 * n, flops=0)   # gathered and scattered: each byte read and written twice
    out_bytes = 4 if case["out"] == "f32" else 2
    Hq, Hkv = case["Hq"], case["Hkv"]
    if op == "prefill":
        chunk, ctx = _prefill_lengths(case)
        pairs = int((chunk * ctx + chunk * (chunk + 1) // 2).sum())
        nt, kv = int(chunk.sum()), int((chunk + ctx).sum())
        b = nt * Hq * D * (2 + out_bytes) + kv * 2 * Hkv * D * 2
        if case["write"]:
            b += 2 * nt * 2 * Hkv * D * 2
        return dict(bytes=b, flops=4 * D * Hq * pairs)
    w, lens = _lengths(case)
    P, S = lens.prefix_lens.astype(np.int64), lens.suffix_lens.astype(np.int64)
    tokens = int(P.sum() + S.sum())
    per_seq = int(S.sum() + P[lens.group_of_seq].sum())
    b = tokens * 2 * Hkv * D * 2 + len(S) * Hq * D * (2 + out_bytes)
    if op == "step":
        n = len(S) * case["vocab"]
        return dict(bytes=b + 2 * n + 2 * len(S) * 2 * Hkv * D * 2, flops=4 * D * Hq * per_seq + 3 * n)
    return dict(bytes=b, flops=4 * D * Hq * per_seq)


def tolerance(case):
    """About four times what two correct orders of summation show (other chunk sizes; the 64-bit result).

    Attention multiplies softmax weights rounded to bf16 with bf16 values: 1.5e-3 (float32 output) to
    2.3e-3 (bf16 output) from the 64-bit result, single values up to 1.3e-2 of it, in a prompt's first
    rows, which average few values, 3.9e-2.  Log-probabilities are float32 sums: 8e-8."""
    op = case["op"]
    if op == "pack":
        return "exact"
    if op in ("logprobs", "sample", "top_p"):
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}
    rel = 7e-3 if case["out"] == "f32" else 9e-3
    return {"rel": rel, "max": 0.15 if op == "prefill" else 0.05, "differ": 1e-3}


# ---- the same in 64 bits -----------------------------------------------------------------------
def _pages_of(pages, row, n):
    """The first n tokens of a block-table row as float64: keys or values [Hkv, n, D]."""
    ids = row[: (n + PAGE - 1) // PAGE].long()
    x = pages[ids]
    x = x.permute(1, 0, 2, 3) if x.shape[2] == PAGE else x.permute(1, 0, 3, 2)
    return x.reshape(x.shape[0], -1, D)[:, :n].double()


def _exact_attn(inp, k_pages, v_pages, suffix_lens):
    NS, Hq, Hkv = inp.num_seqs, inp.Hq, inp.Hkv
    R = Hq // Hkv
    out = torch.zeros(NS, Hq, D, dtype=torch.float64, device="cuda")
    gos, P, S = inp.group_of_seq.cpu().numpy(), inp.prefix_lens.tolist(), suffix_lens.tolist()
    for g in range(inp.num_groups):
        members = np.nonzero(gos == g)[0]
        if len(members) == 0:
            continue
        kp, vp = (_pages_of(x, inp.prefix_block_table[g], P[g]) for x in (k_pages, v_pages))
        for s in members.tolist():
            q = inp.q[s].double().view(Hkv, R, D)
            ks, vs = (_pages_of(x, inp.suffix_block_table[s], S[s]) for x in (k_pages, v_pages))
            x = torch.cat([q @ kp.transpose(1, 2), q @ ks.transpose(1, 2)], 2) * inp.scale
            p = torch.softmax(x, 2)
            out[s] = (p[:, :, : P[g]] @ vp + p[:, :, P[g]:] @ vs).reshape(Hq, D)
    return out


def _exact_prefill(inp, k_pages, v_pages):
    R = inp.Hq // inp.Hkv
    out = torch.zeros(inp.num_tokens, inp.Hq, D, dtype=torch.float64, device="cuda")
    start, pos0 = inp.q_start.tolist(), inp.q_pos0.tolist()
    for g in range(inp.num_groups):
        n, p0 = start[g + 1] - start[g], pos0[g]
        k, v = (_pages_of(x, inp.prefix_block_table[g], p0 + n) for x in (k_pages, v_pages))
        hidden = torch.arange(p0 + n, device="cuda")[None, :] > torch.arange(p0, p0 + n, device="cuda")[:, None]
        for h in range(inp.Hq):
            q = inp.q[start[g]:start[g + 1], h].double()
            x = (q @ k[h // R].t() * inp.scale).masked_fill_(hidden, -math.inf)
            out[start[g]:start[g + 1], h] = torch.softmax(x, 1) @ v[h // R]
    return out


def _scatter_prompt(inp):
    k, v = inp.k_pages.clone(), inp.v_pages.clone()
    start, pos0 = inp.q_start.tolist(), inp.q_pos0.tolist()
    for g in range(inp.num_groups):
        pos = torch.arange(pos0[g], pos0[g] + start[g + 1] - start[g], device="cuda")
        page = inp.prefix_block_table[g][pos // PAGE].long()
        k[page, :, pos % PAGE, :] = inp.k_new[start[g]:start[g + 1]]
        v[page, :, :, pos % PAGE] = inp.v_new[start[g]:start[g + 1]]
    return k, v


def exact(case, seed):
    op = case["op"]
    if op == "pack":
        return None   # bytes, not computed numbers
    s = prepare(case, seed)
    if op == "decode":
        return _exact_attn(s["inp"], s["inp"].k_pages, s["inp"].v_pages, s["inp"].suffix_lens)
    if op == "prefill":
        if not case["write"]:
            return _exact_prefill(s["inp"], s["inp"].k_pages, s["inp"].v_pages)
        k, v = _scatter_prompt(s["inp"])
        return dict(out=_exact_prefill(s["inp"], k, v), k=None, v=None)
    if op == "logprobs":
        rows, vocab = s["logits"].shape
        out = torch.empty(rows, dtype=torch.float64, device="cuda")
        step = max(1, (1 << 27) // vocab)
        for a in range(0, rows, step):
            x = s["logits"][a:a + step].double() / case["T"]
            out[a:a + step] = x.gather(1, s["tokens"][a:a + step, None].long())[:, 0] - torch.logsumexp(x, 1)
        return out
    gen_seed = seed + 2 if op == "step" else seed
    logits, gen = _logits(s["logits"].shape[0], case["vocab"], case["sigma"], gen_seed)
    _, _, lp = _draw_uniforms(logits, case["T"], case.get("top_p", 1.0), gen)
    if op != "step":
        return dict(tokens=None, logprobs=lp)
    inp = s["inp"]
    pos = s["lens_now"].long()
    page = inp.suffix_block_table.gather(1, (pos // PAGE)[:, None])[:, 0].long()
    k, v = inp.k_pages.clone(), inp.v_pages.clone()
    k[page, :, pos % PAGE, :] = s["k_new"]
    v[page, :, :, pos % PAGE] = s["v_new"]
    return dict(out=_exact_attn(inp, k, v, inp.suffix_lens), tokens=None, logprobs=lp, lens=None, k=None, v=None)
