"""The performance cases of libspecverify: calls of a draft-verify round as a serving engine
makes them, through paper_2607_25852_amd.binding, with their inputs, work and 64-bit results.

Interface: listed(), draw(rng), prepare(case, seed), run(state), work(case),
tolerance(case), exact(case, seed).

A case is a dict of plain values:
  op      "prepare"  sv_prepare_round (budget, packing, attention plan), cost-table budget
          "append"   sv_append_kv of the kept rows
          "attn"     sv_verify_attn_run on the round's plan (one layer of the target model)
          "accept"   sv_spec_accept: bf16 or fp32 logits, probability rows (probs), or greedy
                     verification (temperature 0)
          "drafter"  sv_draft_stats over the draft rows, then sv_spec_accept_stats
          "round"    the round's set-up, one attention layer and acceptance
  R, b    concurrent requests, block positions per request (certain token + drafts)
  keep    the share of the R*b positions that is verified, in permille (at least R positions)
  ctx, ctx_lo, ctx_hi   committed context lengths: lognormal with median ctx and sigma 1
          clipped to [ctx_lo, ctx_hi], or uniform over [ctx_lo, ctx_hi] when ctx is 0
  Hq, Hkv, d, page      heads, head dim and page size of the bf16 paged cache
  V, dtype, temperature, probs   vocabulary, logit type and acceptance mode
The lengths are the quantiles of their distribution in a seeded order, so the bytes of a
case do not depend on the seed.
"""
import math
import statistics

import torch

from paper_2607_25852_amd import binding as B
from paper_2607_25852_amd import synth

# per-request difficulty classes: (draft noise sigma, range of the target's peak mass)
CLASSES = synth.CLASSES
RATIOS = synth.PAPER_RATIOS_PM
HEADS64 = dict(Hq=64, Hkv=8, d=128, page=64)


def listed():
    return [
        # The set-up of the smallest round: four users, a multi-token-prediction head of depth
        # 4. Latency of one launch.
        dict(name="prepare_mtp_c4", op="prepare", R=4, b=5, ctx=8192, ctx_lo=512, ctx_hi=65536, **HEADS64),
        # The set-up of a full round: 64 requests with 16-position blocks.
        dict(name="prepare_blk_c64", op="prepare", R=64, b=16, ctx=4096, ctx_lo=512, ctx_hi=32768, **HEADS64),
        # Once per layer: the kept rows' keys and values into the paged cache.
        dict(name="append_blk_c64", op="append", R=64, b=16, keep=500, ctx=4096, ctx_lo=512, ctx_hi=32768, **HEADS64),
        # Attention at low concurrency: few requests, short blocks, mixed contexts.
        dict(name="attn_mtp_c4", op="attn", R=4, b=5, keep=1000, ctx=8192, ctx_lo=512, ctx_hi=65536, **HEADS64),
        # A smaller model with 64-wide heads on 16-token pages (the common page size of serving
        # engines), odd concurrency and an 8-position block.
        dict(name="attn_page16_c27", op="attn", R=27, b=8, keep=600, ctx=0, ctx_lo=1000, ctx_hi=8191,
             Hq=32, Hkv=8, d=64, page=16),
        # Long contexts: 64K to 128K tokens per request, 16 query heads per kv-head. The largest.
        dict(name="attn_long_c32", op="attn", R=32, b=16, keep=520, ctx=0, ctx_lo=65536, ctx_hi=131072,
             Hq=64, Hkv=4, d=128, page=64),
        # Acceptance at low concurrency: 36 rows of a 131072-token vocabulary.
        dict(name="accept_mtp_c4", op="accept", R=4, b=5, keep=1000, V=131072, dtype="bf16", temperature=1.0,
             probs=False),
        # A sampler that keeps fp32 logits, an odd vocabulary and a temperature below one.
        dict(name="accept_f32_odd_c16", op="accept", R=16, b=8, keep=700, V=50257, dtype="f32", temperature=0.7,
             probs=False),
        # Probability rows handed over by a sampler (after top-p, say) instead of logits.
        dict(name="accept_probs_c16", op="accept", R=16, b=16, keep=1000, V=32768, dtype="f32", temperature=1.0,
             probs=True),
        # Greedy verification of a full round (temperature 0): the kept target rows once.
        dict(name="greedy_blk_c64", op="accept", R=64, b=16, keep=500, V=131072, dtype="bf16", temperature=0.0,
             probs=False),
        # The drafter's row statistics and the acceptance that uses them.
        dict(name="drafter_blk_c32", op="drafter", R=32, b=16, keep=500, V=131072, dtype="bf16", temperature=1.0),
        # A whole round: set-up, one attention layer, acceptance.
        dict(name="round_blk_c64", op="round", R=64, b=16, keep=500, ctx=4096, ctx_lo=512, ctx_hi=32768, V=131072,
             dtype="bf16", temperature=1.0, **HEADS64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_heads(rng):
    Hq, Hkv = rng.choice(((32, 8), (64, 8), (64, 4), (32, 4), (28, 4)))
    return dict(Hq=Hq, Hkv=Hkv, d=rng.choice((64, 128, 128)), page=rng.choice((16, 32, 64, 64, 128)))


def _draw_ctx(rng, case, most):
    """Context lengths for `case` whose keys and values take at most `most` bytes."""
    per_tok = 4 * case["Hkv"] * case["d"] * case["R"]
    if rng.random() < 0.5:
        med = min(_log_int(rng, 512, 16384), max(64, most // (2 * per_tok)))
        case.update(ctx=med, ctx_lo=max(1, med // 8), ctx_hi=med * 8)
    else:
        hi = min(_log_int(rng, 1024, 131072), max(128, most // per_tok))
        case.update(ctx=0, ctx_lo=rng.randint(1, hi // 2), ctx_hi=hi)
    return case


def draw(rng):
    op = rng.choice(("prepare", "append", "attn", "attn", "attn", "accept", "accept", "accept", "drafter", "round"))
    case = dict(op=op, R=_log_int(rng, 4, 64), b=rng.choice((5, 5, 8, 16, 16, rng.randint(2, 16))))
    if op == "prepare":
        case["R"] = _log_int(rng, 4, 512)
    else:
        case["keep"] = rng.choice((250, 500, 500, 750, 1000))
    if op in ("prepare", "append", "attn", "round"):
        case.update(_draw_heads(rng))
        if op == "prepare" and (case["Hq"] // case["Hkv"]) * case["b"] > 1024:
            case["b"] = 5
        _draw_ctx(rng, case, {"append": 1 << 30, "round": 1 << 30}.get(op, 3 << 30))
    if op in ("accept", "drafter", "round"):
        V = _log_int(rng, 32000, 151936)
        V = rng.choice((V // 64 * 64, V // 64 * 64, V // 8 * 8, V | 1))
        case.update(V=V, dtype=rng.choice(("bf16", "bf16", "f32")), temperature=rng.choice((1.0, 1.0, 0.7, 1.3)))
        if op == "accept":
            case["probs"] = rng.random() < 0.25
            if case["probs"]:
                case.update(dtype="f32", temperature=1.0)
            elif rng.random() < 0.25:
                case["temperature"] = 0.0
        elif op == "round":
            case["dtype"] = "bf16"
        if case["dtype"] == "f32":
            case["R"] = min(case["R"], 32)
    return case


# ---------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------
def _lengths(case):
    """The multiset of committed context lengths."""
    R, out = case["R"], []
    for i in range(R):
        x = (i + 0.5) / R
        if case["ctx"]:
            v = case["ctx"] * math.exp(statistics.NormalDist().inv_cdf(x))
        else:
            v = case["ctx_lo"] + x * (case["ctx_hi"] - case["ctx_lo"])
        out.append(int(min(max(round(v), case["ctx_lo"]), case["ctx_hi"])))
    return out


def _budget(case):
    """K: the positions that are verified."""
    R, N = case["R"], case["R"] * case["b"]
    return min(N, max(R, -(-case.get("keep", 500) * N // 1000)))


def _gen(seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))
    return g


def _classes(R, g, dev):
    return (torch.arange(R, device=dev) % len(CLASSES))[torch.randperm(R, generator=g, device=dev)]


def _uniforms(shape, g, dev):
    return torch.randint(0, 1 << 24, shape, generator=g, device=dev).to(torch.float32) * 2.0 ** -24


def _confidences(case, g, dev):
    """[R, b-1] drafter confidences, by the requests' classes."""
    R, D = case["R"], case["b"] - 1
    rng = torch.tensor([[lo, hi] for _, lo, hi in CLASSES], device=dev)[_classes(R, g, dev)]
    return rng[:, :1] + (rng[:, 1:] - rng[:, :1]) * torch.rand((R, D), generator=g, device=dev)


def _logits(case, g, dev):
    """Target rows of every position and draft rows in storage type, draft tokens, confidences."""
    R, b, V = case["R"], case["b"], case["V"]
    D = b - 1
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    target = torch.empty((R, b, V), dtype=dt, device=dev)
    draft = torch.empty((R, D, V), dtype=dt, device=dev)
    tokens = torch.empty((R, D), dtype=torch.int32, device=dev)
    conf = torch.empty((R, D), dtype=torch.float32, device=dev)
    for i, c in enumerate(_classes(R, g, dev).tolist()):
        sigma, lo, hi = CLASSES[c]
        t = torch.randn((b, V), generator=g, device=dev) * 3.0
        tok = torch.randint(0, V, (b, 1), generator=g, device=dev)
        mass = lo + (hi - lo) * torch.rand((b, 1), generator=g, device=dev)
        t.scatter_(1, tok, -math.inf)
        t.scatter_(1, tok, torch.log(mass / (1 - mass)) + torch.logsumexp(t, 1, keepdim=True))
        target[i] = t
        draft[i] = t[:D] + torch.randn((D, V), generator=g, device=dev) * sigma
        p = torch.softmax(draft[i].float(), 1)
        tokens[i] = torch.multinomial(p, 1, generator=g)[:, 0].to(torch.int32)
        conf[i] = p.max(1).values
    return target, draft, tokens, conf


def _keep(s, case, conf, dev):
    """The packing of the kept positions (qo) by the fixed budget."""
    R, b = case["R"], case["b"]
    K = _budget(case)
    keep = torch.empty(R, dtype=torch.int32, device=dev)
    sel = torch.empty(2, dtype=torch.int32, device=dev)
    s["qo"] = torch.empty(R + 1, dtype=torch.int32, device=dev)
    B.alloc_budget(B.budget_desc(R, b, "fixed", fixed_budget=K), conf, keep, s["qo"], sel)
    return s["qo"].cpu().tolist()


def _setup_state(s, case, conf, cost_mode, g, dev):
    """Arguments of sv_prepare_round."""
    R, b = case["R"], case["b"]
    L = torch.tensor(_lengths(case), dtype=torch.int32, device=dev)[torch.randperm(R, generator=g, device=dev)]
    s["ctx"] = L.contiguous()
    s["conf"] = conf.contiguous()
    if cost_mode:
        s["bdesc"] = B.budget_desc(R, b, "cost", ratios_pm=RATIOS, cost=synth.profiled_cost(R, b))
    else:
        s["bdesc"] = B.budget_desc(R, b, "fixed", fixed_budget=_budget(case))
    i32 = dict(dtype=torch.int32, device=dev)
    s.update(keep=torch.zeros(R, **i32), qo=torch.zeros(R + 1, **i32), sel=torch.zeros(2, **i32),
             scores=torch.zeros((R, b), device=dev),
             util=torch.zeros(len(RATIOS) if cost_mode else 1, dtype=torch.int64, device=dev),
             pdesc=B.pack_desc(R, b, R * b), block_tokens=torch.randint(0, 131072, (R, b), generator=g, **i32),
             v_tokens=torch.zeros(R * b, **i32), v_positions=torch.zeros(R * b, **i32), kv_lens=torch.zeros(R, **i32))
    need = [-(-(n + b) // case["page"]) for n in L.tolist()]
    pool = int(math.ceil(sum(need) * 1.25))
    pages = torch.randperm(pool, generator=g, device=dev).to(torch.int32)
    pt = torch.full((R, max(need)), -1, **i32)
    at = 0
    for i, n in enumerate(need):
        pt[i, :n] = pages[at:at + n]
        at += n
    s["page_table"] = pt
    s["adesc"] = B.attn_desc(R, R * b, b, case["Hq"], case["Hkv"], case["d"], case["page"], max(need), pool,
                             max(_lengths(case)) + b, B.SV_BF16)
    s["attn_ws"] = torch.empty(max(B.attn_workspace_size(s["adesc"]), 256), dtype=torch.uint8, device=dev)
    return pool


def _attn_state(s, case, pool, g, dev):
    R, b, Hq, Hkv, d, P = (case[k] for k in ("R", "b", "Hq", "Hkv", "d", "page"))
    bf = dict(dtype=torch.bfloat16, device=dev)
    s["k_cache"] = torch.randn((pool, Hkv, P, d), generator=g, **bf)
    s["v_cache"] = torch.randn((pool, Hkv, P, d), generator=g, **bf)
    s["q"] = torch.randn((R * b, Hq, d), generator=g, **bf)
    s["attn_out"] = torch.zeros((R * b, Hq, d), **bf)
    s["attn_lse"] = torch.zeros((R * b, Hq), device=dev)


def _accept_state(s, case, target, draft, tokens, qo, g, dev):
    R, b, V = case["R"], case["b"], case["V"]
    if case.get("probs"):
        target, draft = torch.softmax(target.float(), 2), torch.softmax(draft.float(), 2)
    s["target"] = torch.cat([target[i, :qo[i + 1] - qo[i]] for i in range(R)]).contiguous()
    s["draft"], s["tokens"] = draft, tokens
    s["u_accept"], s["u_sample"] = _uniforms((R, b - 1), g, dev), _uniforms((R,), g, dev)
    dt = B.SV_F32 if case["dtype"] == "f32" else B.SV_BF16
    s["xdesc"] = B.accept_desc(R, b, V, B.SV_PROBS if case.get("probs") else B.SV_LOGITS, dt, case["temperature"])
    i32 = dict(dtype=torch.int32, device=dev)
    s.update(accept_len=torch.zeros(R, **i32), out_tokens=torch.zeros((R, b), **i32), flags=torch.zeros(R, **i32),
             acc_ws=torch.empty(B.accept_workspace_size(s["xdesc"]), dtype=torch.uint8, device=dev))
    if case["op"] == "drafter":
        s["sdesc"] = B.draft_stats_desc(R, b - 1, V, dt, case["temperature"])
        s["stats"] = torch.zeros((R, b - 1, 2), device=dev)
        s["conf"] = torch.zeros((R, b - 1), device=dev)
        s["stats_ws"] = torch.empty(B.draft_stats_workspace_size(s["sdesc"]), dtype=torch.uint8, device=dev)


def prepare(case, seed):
    dev, op = "cuda", case["op"]
    g = _gen(seed, dev)
    s = {"op": op}
    if op in ("accept", "drafter"):
        target, draft, tokens, conf = _logits(case, g, dev)
        qo = _keep(s, case, conf, dev)
        _accept_state(s, case, target, draft, tokens, qo, g, dev)
        return s
    logits = _logits(case, g, dev) if op == "round" else None
    conf = logits[3] if logits else _confidences(case, g, dev)
    pool = _setup_state(s, case, conf, op == "prepare", g, dev)
    if op == "prepare":
        return s
    if op == "append":
        R, b, Hkv, d, P = (case[k] for k in ("R", "b", "Hkv", "d", "page"))
        _keep(s, case, conf, dev)
        bf = dict(dtype=torch.bfloat16, device=dev)
        s["xk"], s["xv"] = (torch.randn((R * b, Hkv, d), generator=g, **bf) for _ in range(2))
        s["k_cache"], s["v_cache"] = (torch.zeros((pool, Hkv, P, d), **bf) for _ in range(2))
        s["apdesc"] = B.append_desc(R, R * b, b, Hkv, d, P, s["page_table"].shape[1], pool, B.SV_BF16)
        return s
    _attn_state(s, case, pool, g, dev)
    if op == "attn":  # a layer of the round: the set-up has run
        _run_prepare(s)
        return s
    qo = _keep({}, case, conf, dev)
    _accept_state(s, case, logits[0], logits[1], logits[2], qo, g, dev)
    s["block_tokens"][:, 1:] = logits[2]
    return s


# ---------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------
def _run_prepare(s):
    B.prepare_round(s["bdesc"], s["conf"], s["keep"], s["qo"], s["sel"], s["scores"], s["util"], s["pdesc"],
                    s["block_tokens"], s["ctx"], s["v_tokens"], s["v_positions"], s["kv_lens"], s["adesc"],
                    s["attn_ws"])


def _run_attn(s):
    B.verify_attn_run(s["adesc"], s["q"], s["k_cache"], s["v_cache"], s["page_table"], s["qo"], s["kv_lens"],
                      s["attn_out"], s["attn_lse"], s["attn_ws"])


def _run_accept(s):
    B.spec_accept(s["xdesc"], s["target"], s["draft"], s["tokens"], s["qo"], s["u_accept"], s["u_sample"],
                  s["accept_len"], s["out_tokens"], s["flags"], s["acc_ws"])


_PREP = ("keep", "qo", "sel", "scores", "util", "v_tokens", "v_positions", "kv_lens")
_ATTN = ("attn_out", "attn_lse")
_ACC = ("accept_len", "out_tokens", "flags")


def run(s):
    op = s["op"]
    if op == "prepare":
        _run_prepare(s)
        names = _PREP
    elif op == "append":
        B.append_kv(s["apdesc"], s["xk"], s["xv"], s["page_table"], s["qo"], s["ctx"], s["k_cache"], s["v_cache"])
        names = ("k_cache", "v_cache")
    elif op == "attn":
        _run_attn(s)
        names = _ATTN
    elif op == "accept":
        _run_accept(s)
        names = _ACC
    elif op == "drafter":
        B.draft_stats(s["sdesc"], s["draft"], s["stats"], s["conf"], s["stats_ws"])
        B.spec_accept_stats(s["xdesc"], s["target"], s["draft"], s["stats"], s["tokens"], s["qo"], s["u_accept"],
                            s["u_sample"], s["accept_len"], s["out_tokens"], s["flags"], s["acc_ws"])
        names = ("stats", "conf") + _ACC
    else:
        _run_prepare(s)
        _run_attn(s)
        _run_accept(s)
        names = _PREP + _ATTN + _ACC
    return {n: s[n] for n in names}


# ---------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------
def work(case):
    R, b, op = case["R"], case["b"], case["op"]
    N, K = R * b, _budget(case)
    nbytes = flops = 0
    if op in ("prepare", "round"):  # confidences, tokens, lengths; depths, packing, scores, the batch
        nbytes += 4 * (R * (b - 1) + N + R) + 4 * (3 * R + N + 2 * K)
    if op == "append":
        nbytes += 2 * 2 * K * case["Hkv"] * case["d"] * 2
    if op in ("attn", "round"):
        L, Hq, d = sum(_lengths(case)), case["Hq"], case["d"]
        nbytes += (L + K) * 2 * case["Hkv"] * d * 2 + K * Hq * (2 * d * 2 + 4)
        flops += 4 * d * Hq * K * (L / R + K / R / 2)
    if op in ("accept", "drafter", "round"):
        row = case["V"] * (4 if case["dtype"] == "f32" else 2)
        rows = K if case["temperature"] == 0 else K + (N - R if op == "drafter" else K - R)
        if case.get("probs"):  # a probability row is read at its drafted token; one pair of rows is drawn from
            rows = 2 * R
        nbytes += rows * row
        flops += 4 * rows * case["V"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Attention: bf16 results and bf16 probabilities under fp32 sums, measured 2.3e-3 off the
    64-bit result. Row statistics: fp32 sums of V exponentials, measured up to 2e-7 off. A token
    drawn where the cumulative sum meets the threshold may differ by the rounding of the sum."""
    op = case["op"]
    if op in ("prepare", "append") or (op == "accept" and (case["probs"] or case["temperature"] == 0)):
        return "exact"
    if op == "attn":
        return {"rel": 1e-2, "max": 0.2}
    if op == "round":
        return {"rel": 1e-2, "max": 0.2, "differ": 0.01}
    return {"rel": 2e-6, "max": 2e-5, "differ": 0.01}


# ---------------------------------------------------------------------------------------
# 64-bit results
# ---------------------------------------------------------------------------------------
def _exact_scores(conf, b):
    c = conf.double().clamp(0, 1)
    return torch.cat([torch.ones_like(c[:, :1]), torch.cumprod(c, 1)], 1)[:, :b]


def _exact_attn(s, case, qo):
    Hq, Hkv, d = case["Hq"], case["Hkv"], case["d"]
    G = Hq // Hkv
    out = torch.zeros(s["q"].shape, dtype=torch.float64, device=s["q"].device)
    lse = torch.zeros(s["q"].shape[:2], dtype=torch.float64, device=s["q"].device)
    for i, L in enumerate(s["ctx"].tolist()):
        q0, k = qo[i], qo[i + 1] - qo[i]
        n = L + k
        pages = s["page_table"][i, :-(-n // case["page"])].long()
        kk, vv = (c[pages].transpose(0, 1).reshape(Hkv, -1, d)[:, :n].double() for c in (s["k_cache"], s["v_cache"]))
        q = s["q"][q0:q0 + k].double().reshape(k, Hkv, G, d).permute(1, 2, 0, 3).reshape(Hkv, G * k, d)
        z = torch.bmm(q, kk.transpose(1, 2).contiguous()) / math.sqrt(d)
        hide = torch.arange(n, device=z.device)[None, :] > L + torch.arange(k, device=z.device)[:, None]
        z.view(Hkv, G, k, n).masked_fill_(hide, -math.inf)
        ls = torch.logsumexp(z, 2)
        o = torch.bmm(torch.exp_(z.sub_(ls[:, :, None])), vv)
        out[q0:q0 + k] = o.view(Hkv, G, k, d).permute(2, 0, 1, 3).reshape(k, Hq, d)
        lse[q0:q0 + k] = ls.view(Hkv, G, k).permute(2, 0, 1).reshape(k, Hq)
        del z
    return out, lse


def exact(case, seed):
    op = case["op"]
    if op in ("append", "accept"):
        return None  # copies and whole numbers
    s = prepare(case, seed)
    if op == "prepare":
        return dict({n: None for n in _PREP}, scores=_exact_scores(s["conf"], case["b"]))
    if op == "drafter":
        x = s["draft"].double() * (1.0 / case["temperature"])
        m = x.amax(2)
        S = torch.exp(x - m[:, :, None]).sum(2)
        return dict({n: None for n in _ACC}, stats=torch.stack([m, S], 2), conf=1 / S)
    if op == "round":
        qo = _keep({}, case, s["conf"], s["conf"].device)
    else:
        qo = s["qo"].cpu().tolist()
    out, lse = _exact_attn(s, case, qo)
    if op == "attn":
        return dict(attn_out=out, attn_lse=lse)
    return dict({n: None for n in _PREP + _ACC}, scores=_exact_scores(s["conf"], case["b"]), attn_out=out, attn_lse=lse)
