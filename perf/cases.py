"""Performance cases of the sdblock library: what one speculative step, and the calls around it,
cost a user on one MI355X, through the public Python entry points.

A case is a dict of plain values.  `listed()` are the named cases, `draw()` makes more of the same
ranges, `prepare()` builds what a caller holds before the call (on the GPU), `run()` is one pass,
`work()` the bytes and operations a pass cannot do without, `exact()` the same outputs in 64 bits
by plain torch and `tolerance()` the error a correct implementation of the same precision shows.

Ragged lengths follow from the case alone (`lens` seeds them), so the work of a case is known
without its inputs; values follow from the seed given to `prepare()`.
"""
import math
import random

import torch

import paper_2606_31315_amd as sd

DEV = "cuda"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
MASKS = {"causal": sd.SD_MASK_CAUSAL_IN_BLOCK, "bidir": sd.SD_MASK_BIDIR_IN_BLOCK}


def _attn(name, S, ctx, block, heads=(32, 8), D=128, dtype="bf16", mask="causal", lens=1, page=0):
    return {"name": name, "op": "attn", "S": S, "Hq": heads[0], "Hkv": heads[1], "D": D, "dtype": dtype,
            "mask": mask, "ctx_lo": ctx[0], "ctx_hi": ctx[1], "b_lo": block[0], "b_hi": block[1], "lens": lens,
            "page": page}


def _accept(name, S, block, V, T, dtype="bf16", lens=1):
    return {"name": name, "op": "accept", "S": S, "b_lo": block[0], "b_hi": block[1], "V": V, "T": T,
            "dtype": dtype, "lens": lens}


def listed():
    return [
        # the smallest verify call: one sequence, one block of the training size, one layer
        _attn("attn_verify_b1", 1, (2048, 2048), (16, 16)),
        # one whole verify step of a small serving batch with adaptive (ragged) blocks: append and
        # attention in every layer, sampling acceptance, commit (4 of a model's layers)
        {"name": "step_ragged_b8", "op": "step", "layers": 4, "S": 8, "Hq": 32, "Hkv": 8, "D": 128, "dtype": "bf16",
         "mask": "causal", "ctx_lo": 4096, "ctx_hi": 4096, "b_lo": 12, "b_hi": 20, "lens": 3, "V": 151936, "T": 1.0},
        # the block-diffusion drafter's pass: bidirectional blocks, contexts of every length
        _attn("attn_drafter_b16", 16, (1024, 8192), (8, 32), mask="bidir", lens=4),
        # long-context serving over a paged cache
        _attn("attn_long_paged_b32", 32, (8192, 32768), (4, 32), lens=5, page=64),
        # a model kept in fp32, odd contexts and blocks
        _attn("attn_fp32_b4", 4, (700, 3001), (7, 21), dtype="f32", lens=6),
        # greedy decoding of the serving batch
        _accept("accept_greedy_b8", 8, (12, 20), 151936, 0.0, lens=3),
        # sampling acceptance of the long-context batch, the largest logits a step brings
        _accept("accept_sample_b32", 32, (4, 32), 151936, 1.0, lens=5),
        # one sequence with fp32 logits over an odd vocabulary (rows not 16-byte aligned)
        _accept("accept_fp32_b1", 1, (12, 12), 50257, 0.7, dtype="f32", lens=7),
        # the block-size policy of one prompt, and of a batch admitted together
        {"name": "policy_p1", "op": "policy", "P": 1, "V": 151936, "H": 2048, "radius": 2, "dtype": "bf16"},
        {"name": "policy_p8", "op": "policy", "P": 8, "V": 151936, "H": 2048, "radius": 2, "dtype": "bf16"},
        # the prefix-survival model over a population of prompts, closed form and Monte Carlo
        {"name": "survival_tau", "op": "tau", "N": 1 << 20, "P": 32, "radius": 2, "alpha": 0.001},
        {"name": "survival_mc", "op": "mc", "N": 1 << 16, "P": 32, "radius": 2, "alpha": 0.001, "trials": 1024},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: batches of 1 to 32 sequences, contexts from a short prompt to
    32k, blocks of 1 to 64 rows, both head sizes, masks and types, contiguous and paged caches."""
    op = rng.choice(["attn", "attn", "attn", "paged", "f32", "step", "accept", "accept", "policy", "tau", "mc"])
    lens = rng.randrange(1 << 20)
    if op in ("attn", "paged", "f32", "step"):
        heads, D = rng.choice([(32, 8), (32, 8), (32, 4), (16, 8), (8, 8)]), rng.choice([128, 128, 64])
        S = _log(rng, 1, 32)
        # no more keys in all than the long-context case (fp32 and whole steps: a tenth)
        top = min(32768, (600_000 if op in ("attn", "paged") else 60_000) // S)
        hi = _log(rng, 200, top)
        lo = max(1, int(hi * rng.uniform(0.2, 1.0)))
        bh = min(_log(rng, 2, 32 if op == "step" else 64), 256 * heads[1] // heads[0])
        bl = max(1, int(bh * rng.uniform(0.2, 1.0)))
        mask = "causal" if op == "step" else rng.choice(["causal", "bidir"])
        page = rng.choice([16, 64, 256]) if op == "paged" else 0
        c = _attn("", S, (lo, hi), (bl, bh), heads, D, "f32" if op == "f32" else "bf16", mask, lens, page)
        if op == "step":
            c.update(op="step", layers=rng.randint(1, 4), V=_log(rng, 8000, 152000), T=rng.choice([0.0, 0.7, 1.0]))
    elif op == "accept":
        bh = _log(rng, 2, 32)
        c = _accept("", _log(rng, 1, 32), (max(1, int(bh * rng.uniform(0.2, 1.0))), bh), _log(rng, 8000, 152000),
                    rng.choice([0.0, 0.7, 1.0]), rng.choice(["bf16", "bf16", "f32"]), lens)
    elif op == "policy":
        c = {"name": "", "op": "policy", "P": _log(rng, 1, 16), "V": 8 * _log(rng, 1000, 19000),
             "H": 8 * _log(rng, 64, 256), "radius": rng.randint(1, 4), "dtype": rng.choice(["bf16", "f32"])}
    elif op == "tau":
        c = {"name": "", "op": "tau", "N": _log(rng, 1000, 1 << 20), "P": rng.randint(20, 48),
             "radius": rng.randint(1, 4), "alpha": rng.choice([0.0, 0.001, 0.01])}
    else:
        c = {"name": "", "op": "mc", "N": _log(rng, 256, 1 << 15), "P": rng.randint(20, 48),
             "radius": rng.randint(1, 4), "alpha": rng.choice([0.0, 0.001, 0.01]), "trials": _log(rng, 64, 1024)}
    c.pop("name")
    return c


def _lens(case):
    r = random.Random(case["lens"])
    ctx = [r.randint(case.get("ctx_lo", 0), case.get("ctx_hi", 0)) for _ in range(case["S"])]
    blk = [r.randint(case["b_lo"], case["b_hi"]) for _ in range(case["S"])]
    off = [0]
    for b in blk:
        off.append(off[-1] + b)
    return ctx, blk, off


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device=DEV)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _randn(g, shape, dtype, sigma=1.0):
    return torch.randn(shape, generator=g, device=DEV, dtype=dtype) * sigma


# ---- attention ----

def _prepare_attn(case, seed):
    ctx, blk, off = _lens(case)
    g, dt = _gen(seed), DTYPES[case["dtype"]]
    S, Hq, Hkv, D = case["S"], case["Hq"], case["Hkv"], case["D"]
    L = max(ctx) + max(blk)
    st = {"ctx": _i32(ctx), "blk": _i32(blk), "off": _i32(off), "mask": MASKS[case["mask"]], "max_ctx": max(ctx),
          "max_block": max(blk), "q": _randn(g, (off[-1], Hq, D), dt)}
    st["out"] = torch.empty_like(st["q"])
    if case["page"]:
        ps = case["page"]
        n = -(-L // ps)
        pool = S * n + 3
        perm = torch.randperm(pool, generator=torch.Generator().manual_seed(seed))[:S * n]
        st["table"] = perm.to(torch.int32).reshape(S, n).to(DEV)
        st["k"], st["v"] = _randn(g, (pool, Hkv, ps, D), dt), _randn(g, (pool, Hkv, ps, D), dt)
    else:
        st["k"], st["v"] = _randn(g, (S, Hkv, L, D), dt), _randn(g, (S, Hkv, L, D), dt)
    return st


def _run_attn(st):
    kw = dict(max_ctx=st["max_ctx"], max_block=st["max_block"], out=st["out"])
    if "table" in st:
        return sd.block_attn_paged(st["q"], st["k"], st["v"], st["table"], st["ctx"], st["blk"], st["off"],
                                   st["mask"], **kw)
    return sd.block_attn(st["q"], st["k"], st["v"], st["ctx"], st["blk"], st["off"], st["mask"], **kw)


def _attn64(q, ctx, blk, off, causal, rows):
    """Attention of packed ragged blocks in 64 bits; rows(s) gives the sequence's keys and values
    [Hkv, ctx + B, D], the block's own included."""
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    Hq, D = q.shape[1], q.shape[2]
    for s, (c, b) in enumerate(zip(ctx, blk)):
        if b == 0:
            continue
        k, v = rows(s)
        G = Hq // k.shape[0]
        qs = q[off[s]:off[s + 1]].double()
        key, row = torch.arange(c + b, device=q.device), torch.arange(b, device=q.device)
        hide = (key[None, :] > c + row[:, None]).repeat_interleave(G, 0) if causal else None
        for h in range(k.shape[0]):
            qh = qs[:, h * G:(h + 1) * G].reshape(b * G, D)
            w = qh @ k[h].double().t().contiguous() / math.sqrt(D)
            if hide is not None:
                w.masked_fill_(hide, float("-inf"))
            out[off[s]:off[s + 1], h * G:(h + 1) * G] = (torch.softmax(w, 1) @ v[h].double()).reshape(b, G, D)
    return out


def _exact_attn(case, seed):
    st = _prepare_attn(case, seed)
    ctx, blk, off = _lens(case)

    def rows(s):
        n = ctx[s] + blk[s]
        if case["page"]:
            t = st["table"][s].long()
            flat = [x[t].transpose(0, 1).reshape(case["Hkv"], -1, case["D"])[:, :n] for x in (st["k"], st["v"])]
            return flat
        return st["k"][s, :, :n], st["v"][s, :, :n]

    return _attn64(st["q"], ctx, blk, off, case["mask"] == "causal", rows)


# ---- acceptance ----

def _prepare_accept(case, seed):
    _, blk, off = _lens(case)
    g, dt = _gen(seed + 7), DTYPES[case["dtype"]]
    S, V, T, n = case["S"], case["V"], case["T"], off[-1]
    target = _randn(g, (n, V), torch.float32, 3.0).to(dt)
    first = torch.tensor([r for s in range(S) for r in range(off[s], off[s + 1] - 1)], dtype=torch.long, device=DEV)
    draft = (target[first].float() + _randn(g, (len(first), V), torch.float32)).to(dt)
    noisy = draft.float()
    if T > 0:  # Gumbel-max: drawn from the drafter's softmax at this temperature
        u = torch.rand(draft.shape, generator=g, device=DEV).clamp_(1e-9, 1 - 1e-7)
        noisy = noisy / T - torch.log(-torch.log(u))
    tokens = noisy.argmax(1).to(torch.int32) if len(first) else torch.zeros(0, dtype=torch.int32, device=DEV)
    return {"target": target, "draft": draft if T > 0 and len(first) else None, "tokens": tokens,
            "u": torch.rand(n, generator=g, device=DEV) if T > 0 else None, "blk": _i32(blk),
            "off": _i32(off), "T": T, "max_block": max(blk),
            "al": torch.empty(S, dtype=torch.int32, device=DEV), "nt": torch.empty(S, dtype=torch.int32, device=DEV)}


def _run_accept(st):
    return sd.accept(st["target"], st["draft"], st["tokens"], st["u"], st["blk"], st["off"], st["T"],
                     max_block=st["max_block"], accept_len=st["al"], next_token=st["nt"])


# ---- one verify step: every layer's append and attention, acceptance, commit ----

def _prepare_step(case, seed):
    ctx, blk, off = _lens(case)
    g, dt = _gen(seed), DTYPES[case["dtype"]]
    S, Hq, Hkv, D, n = case["S"], case["Hq"], case["Hkv"], case["D"], off[-1]
    L = max(ctx) + max(blk)
    st = _prepare_accept(case, seed)
    st.update(ctx0=_i32(ctx), ctx=_i32(ctx), mask=MASKS[case["mask"]], max_ctx=max(ctx), layers=[])
    for _ in range(case["layers"]):
        q = _randn(g, (n, Hq, D), dt)
        st["layers"].append({"q": q, "k_new": _randn(g, (n, Hkv, D), dt), "v_new": _randn(g, (n, Hkv, D), dt),
                             "k_cache": _randn(g, (S, Hkv, L, D), dt), "v_cache": _randn(g, (S, Hkv, L, D), dt),
                             "out": torch.empty_like(q)})
    return st


def _run_step(st):
    # the step advances ctx in place; start each pass from the same committed lengths
    st["ctx"].copy_(st["ctx0"])
    al, nt = sd.verify_step(st["layers"], st["ctx"], st["blk"], st["off"], st["mask"], st["target"], st["draft"],
                            st["tokens"], st["u"], st["T"], max_ctx=st["max_ctx"], max_block=st["max_block"],
                            accept_len=st["al"], next_token=st["nt"])
    return {"out": [x["out"] for x in st["layers"]], "k": [x["k_cache"] for x in st["layers"]],
            "v": [x["v_cache"] for x in st["layers"]], "accept_len": al, "next_token": nt, "ctx": st["ctx"]}


def _exact_step(case, seed):
    st = _prepare_step(case, seed)
    ctx, blk, off = _lens(case)
    outs = []
    for x in st["layers"]:
        def rows(s, x=x):
            return [torch.cat((x[c][s, :, :ctx[s]], x[n][off[s]:off[s + 1]].transpose(0, 1)), 1)
                    for c, n in (("k_cache", "k_new"), ("v_cache", "v_new"))]
        outs.append(_attn64(x["q"], ctx, blk, off, case["mask"] == "causal", rows))
    return {"out": outs, "k": None, "v": None, "accept_len": None, "next_token": None, "ctx": None}


# ---- the block-size policy ----

def _prepare_policy(case, seed):
    g = _gen(seed)
    P, V, H, C = case["P"], case["V"], case["H"], 2 * case["radius"] + 1
    bf = torch.bfloat16
    return {"logits": _randn(g, (P, V), torch.float32, 3.0).to(DTYPES[case["dtype"]]), "w1": _randn(g, (H, V), bf),
            "b1": _randn(g, (H,), torch.float32, 0.05), "w2": _randn(g, (H, H), bf, H ** -0.5),
            "b2": _randn(g, (H,), torch.float32, 0.05), "w3": _randn(g, (C, H), bf, H ** -0.5),
            "b3": _randn(g, (C,), torch.float32, 0.05),
            "scores": torch.empty(P, C, dtype=torch.float32, device=DEV),
            "size": torch.empty(P, dtype=torch.int32, device=DEV)}


def _run_policy(st):
    return sd.block_size_policy(st["logits"], st["w1"], st["b1"], st["w2"], st["b2"], st["w3"], st["b3"], 16,
                                scores=st["scores"], block_size=st["size"])


def _exact_policy(case, seed):
    st = _prepare_policy(case, seed)
    p = torch.softmax(st["logits"].double(), 1)
    h = torch.cat([w.double() @ p.t().contiguous() for w in st["w1"].split(256)]).t() + st["b1"].double()
    h = torch.relu(torch.relu(h) @ st["w2"].double().t().contiguous() + st["b2"].double())
    return h @ st["w3"].double().t().contiguous() + st["b3"].double(), None


# ---- the prefix-survival model ----

def _prepare_survival(case, seed):
    g = _gen(seed)
    N, P, k = case["N"], case["P"], case["radius"]
    base = 0.6 + 0.37 * torch.rand((N, 1), generator=g, device=DEV)
    gamma = (base + 0.03 * _randn(g, (N, P), torch.float32)).clamp_(0.01, 1.0)
    cands = list(range(16 - k, 16 + k + 1))
    hat = torch.randint(16 - k, 16 + k + 1, (N,), generator=g, device=DEV, dtype=torch.int32)
    return {"gamma": gamma, "cands": cands, "alpha": case["alpha"], "hat": hat, "seed": seed,
            "trials": case.get("trials", 0)}


def _run_survival(st):
    if st["trials"]:
        return sd.survival_sample(st["gamma"], st["cands"], 16, st["alpha"], st["seed"], st["trials"])
    return sd.survival_tau(st["gamma"], st["cands"], 16, st["alpha"], st["hat"])


def _exact_tau(case, seed):
    st = _prepare_survival(case, seed)
    g = st["gamma"].double()
    tau = torch.stack([torch.cumprod(g[:, :b] * math.exp(-st["alpha"] * (b - 16) ** 2), 1).sum(1)
                       for b in st["cands"]], 1)
    hat = tau.gather(1, (st["hat"].long() - st["cands"][0])[:, None])[:, 0]
    return tau, None, tau.max(1).values - hat, (tau[:, 1:] - tau[:, :-1]).abs().max(1).values


_PREPARE = {"attn": _prepare_attn, "accept": _prepare_accept, "step": _prepare_step, "policy": _prepare_policy,
            "tau": _prepare_survival, "mc": _prepare_survival}
_RUN = {"attn": _run_attn, "accept": _run_accept, "step": _run_step, "policy": _run_policy, "tau": _run_survival,
        "mc": _run_survival}
_EXACT = {"attn": _exact_attn, "step": _exact_step, "policy": _exact_policy, "tau": _exact_tau}


def prepare(case, seed):
    st = _PREPARE[case["op"]](case, seed)
    st["op"] = case["op"]
    return st


def run(state):
    return _RUN[state["op"]](state)


def exact(case, seed):
    # acceptance returns whole numbers, and the Monte Carlo means are whole sums over the trials
    f = _EXACT.get(case["op"])
    return f(case, seed) if f else None


def _work_attn(case):
    ctx, blk, _ = _lens(case)
    e = 2 if case["dtype"] == "bf16" else 4
    keys, rows = sum(c + b for c, b in zip(ctx, blk)), sum(blk)
    nbytes = 2 * keys * case["Hkv"] * case["D"] * e + 2 * rows * case["Hq"] * case["D"] * e
    flops = 4 * case["D"] * case["Hq"] * sum(b * (c + b) for c, b in zip(ctx, blk))
    return nbytes, flops


def _work_accept(case):
    _, blk, _ = _lens(case)
    rows = sum(blk) + (sum(blk) - case["S"] if case["T"] > 0 else 0)
    n = rows * case["V"]
    return n * (2 if case["dtype"] == "bf16" else 4), n * (4 if case["T"] > 0 else 1)


def work(case):
    op = case["op"]
    if op == "attn":
        b, f = _work_attn(case)
    elif op == "accept":
        b, f = _work_accept(case)
    elif op == "step":
        b, f = _work_attn(case)
        new = 4 * sum(_lens(case)[1]) * case["Hkv"] * case["D"] * 2  # new rows read and written, K and V
        (ab, af), n = _work_accept(case), case["layers"]
        # the block's keys are counted among the cache rows: the new rows stand in for them
        b, f = n * (b + new // 2) + ab, n * f + af
    elif op == "policy":
        P, V, H, C = case["P"], case["V"], case["H"], 2 * case["radius"] + 1
        b = 2 * (H * V + H * H + C * H) + P * V * (2 if case["dtype"] == "bf16" else 4)
        f = 2 * P * (H * V + H * H + C * H) + 4 * P * V
    else:
        N, P, C = case["N"], case["P"], 2 * case["radius"] + 1
        mean_b = 16
        if op == "tau":
            b, f = N * (4 * P + 4 + 8 * C + 4 + 8 + 8), N * C * mean_b * 3
        else:
            # about 1.7 blocks of four draws per trial (mean accepted length 4 to 5 of these
            # samples), each 20 products of 64 x 64 bits (8 32-bit operations) and 80 of other kinds
            b, f = N * (4 * P + 8 * C + 4 * C * (P + 1)), N * C * case["trials"] * 1.7 * 240
    return {"bytes": b, "flops": f}


def tolerance(case):
    op = case["op"]
    if op in ("attn", "step"):
        # bf16: the output's rounding and the weights' before they meet the values; f32: sums
        return {"rel": 1e-2, "max": 0.1} if case["dtype"] == "bf16" else {"rel": 4e-6, "max": 4e-5}
    if op == "policy":
        return {"rel": 2e-6, "max": 4e-5, "differ": 0.01}
    if op == "tau":
        return {"rel": 3e-14, "max": 1e-12, "differ": 0.001}
    return "exact"  # acceptance decisions and Monte Carlo counts
