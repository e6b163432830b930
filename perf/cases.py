"""The calls this library is measured by: draft verification (and the drafting step's sampling) over the range of
batches, draft lengths, vocabularies and input forms that a serving stack or an experiment hands over.

A case is one call of a public entry point on inputs that live on the GPU, with the workspace and the output buffers a
caller keeps.  Shapes are the library's own workload configurations (B = 1 ... 1024, gamma = 4 ... 16, V = 1000 ...
256000, float32 and bfloat16), the toy models of its outer loop, and the odd or padded vocabularies that real
tokenisers have.

Inputs follow the workloads' recipe: target logits sigma_target * N(0, 1), with or without a Zipf-shaped bias over the
vocabulary, draft logits = target + sigma_draft * N(0, 1), both rounded to the input type, drafted tokens sampled from the
draft distribution, uniforms that are multiples of 2^-24 in [0, 1).
"""
from __future__ import annotations

import math

import torch

import paper_2403_10444_amd as sv

DEVICE = "cuda:0"
TYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
CHUNK_BYTES = 2 << 30            # temporaries while inputs (or exact results) are made


def _case(name, entry, algo, B, gamma, V, dtype, T, sigma_target, sigma_draft, zipf=False, pad=0, ragged=False, debug=False):
    return {"name": name, "entry": entry, "algo": algo, "B": B, "gamma": gamma, "V": V, "dtype": dtype, "T": T,
            "sigma_target": sigma_target, "sigma_draft": sigma_draft, "zipf": zipf, "pad": pad, "ragged": ragged, "debug": debug}


def listed():
    return [
        # one short sequence over a small vocabulary: pure latency
        _case("one_small_f32", "dense", "block", 1, 4, 1000, "f32", 1.0, 2.0, 0.5),
        # the outer loop on toy models: many sequences over a vocabulary of two tokens
        _case("toy_batch_f32", "dense", "block", 8192, 10, 2, "f32", 1.0, 0.5, 0.5),
        # a single stream of decoding with a large vocabulary, on the library's own scratch memory
        _case("one_stream_bf16", "noalloc", "block", 1, 8, 128256, "bf16", 0.8, 4.0, 1.5, zipf=True),
        # a few streams, the baseline algorithm
        _case("few_streams_f32", "dense", "token", 8, 8, 32000, "f32", 1.0, 3.0, 1.0),
        # the same vocabulary at a common batch, with the acceptance probabilities reported for monitoring
        _case("monitored_f32", "dense", "block", 32, 8, 32000, "f32", 1.0, 3.0, 1.0, debug=True),
        # a vocabulary of odd size, as handed over by a language-model head without padding
        _case("odd_vocabulary_bf16", "dense", "token", 24, 4, 50257, "bf16", 1.0, 3.0, 1.0, zipf=True),
        # drafts of different lengths, rows padded for the product that made them, greedy block verification
        _case("ragged_padded_bf16", "ex", "greedy", 48, 6, 100277, "bf16", 0.7, 4.0, 1.0, zipf=True, pad=75, ragged=True),
        # a full serving batch: the headline shape
        _case("serving_batch_bf16", "dense", "block", 64, 8, 128256, "bf16", 0.8, 4.0, 1.5, zipf=True),
        # the same handed over as probabilities
        _case("probabilities_bf16", "probs", "block", 64, 8, 128256, "bf16", 0.8, 4.0, 1.5, zipf=True, debug=True),
        # long drafts of a good drafter at a large batch
        _case("long_drafts_bf16", "dense", "block", 256, 16, 152064, "bf16", 1.0, 4.0, 0.5, zipf=True),
        # the largest batch and vocabulary, sharp distributions
        _case("largest_bf16", "dense", "block", 1024, 8, 256000, "bf16", 0.6, 8.0, 2.0),
        # the drafting step: one token per row for a serving batch
        _case("drafting_bf16", "sample", "sample", 64, 1, 128256, "bf16", 0.8, 4.0, 1.5, zipf=True),
    ]


MOST_LOGITS = 1024 * 17 * 256000            # of one call: the largest listed case


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more call of the same ranges: two in three verify logits, the others take probabilities or draw tokens."""
    entry = rng.choice(["dense", "dense", "ex", "ex", "noalloc", "dense", "ex", "probs", "probs", "sample"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    gamma = 1 if entry == "sample" and rng.random() < 0.5 else rng.randint(1, 16)
    # vocabularies: small experiments now and then, else those of language models; half of them multiples of 64
    V = _log_uniform(rng, 2, 2000) if rng.random() < 0.15 else _log_uniform(rng, 8000, 256000)
    if V > 64 and rng.random() < 0.5:
        V = (V + 63) // 64 * 64
    most = MOST_LOGITS // (4 if dtype == "f32" else 2) // ((2 * gamma + 1) * V)
    if entry == "noalloc":
        # (the library's scratch memory holds calls of this size whatever the split)
        most = min(most, (1 << 31) // ((2 * gamma + 1) * V))
    B = min(_log_uniform(rng, 1, 8192 if V <= 2000 else 1024), max(1, most))
    zipf = rng.random() < 0.5
    ragged = entry in ("ex", "probs") and rng.random() < 0.5
    pad = -V % 64 + rng.choice([0, 64]) if entry in ("ex", "probs") and rng.random() < 0.5 else 0
    algo = "sample" if entry == "sample" else rng.choice(["block", "block", "token", "greedy"])
    # (acceptance is monitored with language models; over a handful of tokens h = S / (S + 1 - w) is often 0 / 0 but for rounding)
    debug = algo in ("block", "token") and V > 2000 and rng.random() < 0.25
    case = _case("", entry, algo, B, gamma, V, dtype, rng.choice([0.6, 0.8, 1.0]), rng.choice([2.0, 3.0, 4.0, 6.0]),
                 rng.choice([0.5, 1.0, 1.5, 3.0]), zipf=zipf, pad=pad, ragged=ragged, debug=debug)
    del case["name"]
    return case


def _uniforms(gen, shape):
    return torch.randint(0, 1 << 24, shape, generator=gen, device=DEVICE, dtype=torch.int32).to(torch.float32) * 2.0 ** -24


def _inputs(case, seed):
    """The call's inputs, from the seed alone."""
    B, g, V, pad = case["B"], case["gamma"], case["V"], case["pad"]
    dt = TYPES[case["dtype"]]
    gen = torch.Generator(device=DEVICE).manual_seed(1_000_003 * int(seed) + 17)
    sample = case["entry"] == "sample"
    probs = case["entry"] == "probs"
    target = None if sample else torch.zeros((B, g + 1, V + pad), dtype=dt, device=DEVICE)[..., :V]
    draft = torch.zeros((B, g, V + pad), dtype=dt, device=DEVICE)[..., :V]
    tokens = torch.empty((B, g), dtype=torch.int32, device=DEVICE)
    bias = -1.1 * torch.log(torch.randperm(V, generator=gen, device=DEVICE).float() + 1.0) if case["zipf"] else None
    step = max(1, min(B, CHUNK_BYTES // ((2 * g + 1) * V * 24)))
    for b0 in range(0, B, step):
        n = min(B, b0 + step) - b0
        t = torch.randn((n, g + 1, V), generator=gen, device=DEVICE).mul_(case["sigma_target"])
        if bias is not None:
            t.add_(bias)
        d = torch.randn((n, g, V), generator=gen, device=DEVICE).mul_(case["sigma_draft"]).add_(t[:, :g])
        if probs:
            t = torch.softmax(t / case["T"], -1)
            d = torch.softmax(d / case["T"], -1)
        if target is not None:
            target[b0:b0 + n] = t
        draft[b0:b0 + n] = d
        if not sample:
            q = draft[b0:b0 + n].float()
            if not probs:
                q = torch.softmax(q / case["T"], -1)
            tokens[b0:b0 + n] = torch.multinomial(q.view(n * g, V), 1, generator=gen).view(n, g).to(torch.int32)
        del t, d
    lens = torch.randint(1, g + 1, (B,), generator=gen, device=DEVICE, dtype=torch.int32) if case["ragged"] else None
    return {"target": target, "draft": draft, "tokens": tokens, "lens": lens,
            "uniforms": _uniforms(gen, (B, g) if sample else (B, g + 1))}


def prepare(case, seed):
    state = _inputs(case, seed)
    B, g, V = case["B"], case["gamma"], case["V"]
    state.update(entry=case["entry"], algo=case["algo"], T=case["T"], debug=None)
    if case["entry"] == "sample":
        return state
    state["accept_len"] = torch.empty(B, dtype=torch.int32, device=DEVICE)
    state["next_token"] = torch.empty(B, dtype=torch.int32, device=DEVICE)
    if case["debug"]:
        # (positions beyond a sequence's draft are not written)
        state["debug"] = torch.zeros((B, g + 1, 3), dtype=torch.float32, device=DEVICE)
    if case["entry"] != "noalloc":
        state["workspace"] = sv.alloc_workspace(B, g, V, DEVICE)
    return state


DENSE = {"block": sv.spec_verify_block, "token": sv.spec_verify_token, "greedy": sv.spec_verify_greedy}


def run(state):
    s = state
    if s["entry"] == "sample":
        return {"tokens": sv.spec_sample_tokens(s["draft"], s["uniforms"], s["T"], tokens=s["tokens"])}
    if s["entry"] == "dense":
        DENSE[s["algo"]](s["target"], s["draft"], s["tokens"], s["uniforms"], s["T"], workspace=s["workspace"],
                         accept_len=s["accept_len"], next_token=s["next_token"], debug_out=s["debug"])
    elif s["entry"] == "ex":
        sv.spec_verify_ex(s["algo"], s["target"], s["draft"], s["tokens"], s["uniforms"], s["T"], draft_lens=s["lens"],
                          workspace=s["workspace"], accept_len=s["accept_len"], next_token=s["next_token"], debug_out=s["debug"])
    elif s["entry"] == "noalloc":
        sv.spec_verify_ex_noalloc(s["algo"], s["target"], s["draft"], s["tokens"], s["uniforms"], s["T"], s["accept_len"],
                                  s["next_token"], debug_out=s["debug"])
    else:
        sv.spec_verify_probs(s["algo"], s["target"], s["draft"], s["tokens"], s["uniforms"], draft_lens=s["lens"],
                             workspace=s["workspace"], accept_len=s["accept_len"], next_token=s["next_token"], debug_out=s["debug"])
    out = {"accept_len": s["accept_len"], "next_token": s["next_token"]}
    if s["debug"] is not None:
        out["debug"] = s["debug"]
    return out


def work(case):
    """Every logit (probability) read once; per logit a scaling, an exponential and a sum, per pair of rows the residual."""
    B, g, V = case["B"], case["gamma"], case["V"]
    size = 4 if case["dtype"] == "f32" else 2
    if case["entry"] == "sample":
        return {"bytes": B * g * (V * size + 8), "flops": B * g * V * 4}
    used = (g + 1) / 2 if case["ragged"] else g          # draft lengths are uniform over 1 .. gamma
    logits = B * (2 * used + 1) * V
    small = B * (4 * used + 4 * (used + 1) + 8) + (B * (used + 1) * 12 if case["debug"] else 0)
    per_logit = 0 if case["entry"] == "probs" else 4
    return {"bytes": logits * size + small, "flops": logits * per_logit + B * used * V * 3}


def tolerance(case):
    # The reported w, S and h are built on float32 sums of float32 exponentials: against 64 bits up to 4e-7 off, mostly
    # 3e-8.  accept_len and next_token are decisions on a uniform against such sums: a uniform next to an edge may fall to
    # its other side (2 of 66 546 tokens against 64 bits).
    return {"rel": 1.6e-6, "max": 1e-4, "differ": 0.001}


def exact(case, seed):
    x = _inputs(case, seed)
    B, g, V, T = case["B"], case["gamma"], case["V"], case["T"]

    def draws(weights, u):
        """min{x : C_x > u C_total} per row."""
        c = torch.cumsum(weights, -1)
        return torch.searchsorted(c, u.double().unsqueeze(-1) * c[..., -1:], right=True).squeeze(-1).clamp_(max=V - 1).to(torch.int32)

    step = max(1, min(B, CHUNK_BYTES // ((2 * g + 1) * V * 8)))
    if case["entry"] == "sample":
        parts = [draws(torch.softmax(x["draft"][b:b + step].double() / T, -1), x["uniforms"][b:b + step]) for b in range(0, B, step)]
        return {"tokens": torch.cat(parts)}
    probs, algo = case["entry"] == "probs", case["algo"]
    taus, ys, blocks = [], [], []
    for b in range(0, B, step):
        P, Q = x["target"][b:b + step].double(), x["draft"][b:b + step].double()
        tok, u = x["tokens"][b:b + step].long(), x["uniforms"][b:b + step].double()
        n = P.shape[0]
        lens = x["lens"][b:b + step].long() if x["lens"] is not None else torch.full((n,), g, device=DEVICE)
        if probs:
            lr = (P[:, :g].gather(2, tok[..., None]) / Q.gather(2, tok[..., None])).squeeze(-1).log()
        else:
            P.div_(T), Q.div_(T)
            Lp, Lq = torch.logsumexp(P, -1), torch.logsumexp(Q, -1)
            lr = (P[:, :g].gather(2, tok[..., None]) - Q.gather(2, tok[..., None])).squeeze(-1) - Lp[:, :g] + Lq
            P.sub_(Lp[..., None]).exp_(), Q.sub_(Lq[..., None]).exp_()
        lw = [torch.zeros(n, dtype=torch.float64, device=DEVICE)]
        for i in range(g):
            nxt = lw[-1] + lr[:, i]
            lw.append(nxt.clamp(max=0.0) if algo == "block" else nxt)
        lw = torch.zeros((n, g + 1), dtype=torch.float64, device=DEVICE) if algo == "token" else torch.stack(lw, 1)
        w = lw.exp()
        pos = torch.arange(g + 1, device=DEVICE)
        last = pos[None] == lens[:, None]
        S = torch.stack([(w[:, i, None] * P[:, i] - Q[:, i]).clamp_(min=0).sum(-1) for i in range(g)], 1)
        S = torch.cat([S, torch.zeros((n, 1), dtype=torch.float64, device=DEVICE)], 1)
        row_mass = P.gather(1, lens[:, None, None].expand(n, 1, V)).sum(-1) if probs and algo != "block" else 1.0
        S = torch.where(last, w * row_mass, S)
        if algo == "token":
            h = torch.cat([torch.ones((n, 1), dtype=torch.float64, device=DEVICE), lr.clamp(max=0.0).exp()], 1)
        elif algo == "greedy" and probs:
            R = torch.stack([(Q[:, i] - w[:, i, None] * P[:, i]).clamp_(min=0).sum(-1) for i in range(g)], 1)
            h = torch.cat([torch.where(R > 0, S[:, :g] / R, 1.0), w[:, g:]], 1)
        else:
            h = torch.where(w >= 1.0, 1.0, S / (S - torch.expm1(lw.clamp(max=0.0))))
        if algo != "token":
            h = torch.where(last, w, h).clamp_(max=1.0)
        h[:, 0] = 1.0
        passed = (u[:, :g] < h[:, 1:]) & (pos[None, 1:] <= lens[:, None])
        if algo == "token":
            tau = torch.cumprod(passed.long(), 1).sum(1)
        else:
            tau = (passed * pos[None, 1:]).max(1).values
        weights = P.gather(1, tau[:, None, None].expand(n, 1, V)).squeeze(1)
        q = Q.gather(1, tau.clamp(max=g - 1)[:, None, None].expand(n, 1, V)).squeeze(1)
        rest = (w.gather(1, tau[:, None]) * weights - q).clamp_(min=0)
        keep = (tau == lens) | (rest.sum(-1) <= 0)
        weights = torch.where(keep[:, None], weights, rest)
        taus.append(tau.to(torch.int32))
        ys.append(draws(weights, u.gather(1, lens[:, None]).squeeze(1)))
        blocks.append(torch.stack([w, S, h], 2) * (pos[None] <= lens[:, None])[..., None])
    out = {"accept_len": torch.cat(taus), "next_token": torch.cat(ys)}
    if case["debug"]:
        out["debug"] = torch.cat(blocks)
    return out
