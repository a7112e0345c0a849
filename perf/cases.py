"""Performance cases: what a rollout worker asks of the library, one case per kind of call and size.

A case names a call (``call``), the layer's head shape, the batch and the KV type. Lengths are the
quantiles of the case's distribution in an order drawn from the seed, so every seed has the same work
and other data. Pools hold exactly the needed pages, physically permuted.

Calls:
  attention    the decode attention over a batch whose K/V are all cached (``DeviceBatch.attention``)
  append       the KV append of one new token per sequence, then the attention (``DeviceBatch.step``)
  projections  the decode step from the raw projections: q/k norm, rotary embedding, append and plan,
               then partial attention and combine (``qk_prep_plan``, ``attn_parts``, ``combine_parts``)
  prep         the pre-attention side alone, as every layer after the first of a planned step runs it
  prefill      the prompts of a round: K/V pages and causal attention (``PrefillBatch.prefill``)
"""
import math
import random
import statistics

import numpy as np
import torch

import paper_2606_26997_amd as rp

PAGE = 16


def _decode(name, call, *, hq=16, hkv=8, d=128, groups, group_size, prefix, resp, live=0, dtype="bf16", k_mult=1.0):
    """resp: (low, high) uniform, or (median, sigma, cap) log-normal."""
    c = dict(name=name, call=call, hq=hq, hkv=hkv, d=d, groups=groups, group_size=group_size, prefix_lo=prefix[0],
             prefix_hi=prefix[1], live=live, dtype=dtype, k_mult=k_mult)
    if len(resp) == 2:
        c.update(resp_lo=resp[0], resp_hi=resp[1], resp_sigma=0.0)
    else:
        c.update(resp_lo=resp[0], resp_hi=resp[2], resp_sigma=resp[1])
    return c


def _prefill(name, *, hq=16, hkv=8, d=128, groups, prompt, dtype="bf16"):
    return dict(name=name, call="prefill", hq=hq, hkv=hkv, d=d, groups=groups, prefix_lo=prompt[0],
                prefix_hi=prompt[1], dtype=dtype)


def listed():
    return [
        # One small group early in its rollout: the smallest decode call, all latency and launches.
        _decode("decode_tiny", "attention", hq=4, hkv=2, d=64, groups=1, group_size=4, prefix=(128, 128),
                resp=(32, 64)),
        # Frontier-group dispatch: two groups of eight in flight, one layer of the step from the projections.
        _decode("frontier_step", "projections", groups=2, group_size=8, prefix=(512, 512), resp=(0, 6016)),
        # An ordinary batch in mid-rollout: 32 prompts of 8 responses, ragged everywhere.
        _decode("decode_groups", "attention", groups=32, group_size=8, prefix=(64, 512), resp=(0, 4096), k_mult=0.5),
        # A large batch with a long tail of lengths, each step appending a token first.
        _decode("decode_append", "append", groups=64, group_size=16, prefix=(256, 256), resp=(1500.0, 0.9, 8192)),
        # The largest call: long responses, groups partly finished, sequences in no particular order.
        _decode("decode_mixed", "attention", groups=128, group_size=8, prefix=(128, 1024), resp=(0, 16384), live=512),
        # Long contexts in an fp8 cache, with the append and its scale rule.
        _decode("decode_fp8_long", "append", groups=16, group_size=16, prefix=(256, 256), resp=(8192, 32768),
                dtype="fp8"),
        # A layer whose kv-heads each serve eight query heads.
        _decode("decode_ratio8", "attention", hq=32, hkv=4, groups=32, group_size=8, prefix=(64, 512),
                resp=(0, 8192)),
        # A layer with 64-wide heads, four query heads per kv-head.
        _decode("decode_d64", "attention", hq=32, hkv=8, d=64, groups=32, group_size=8, prefix=(64, 512),
                resp=(0, 4096)),
        # The pre-attention side of a large batch with an fp8 cache.
        _decode("prep_fp8", "prep", groups=64, group_size=16, prefix=(256, 256), resp=(0, 2048), dtype="fp8"),
        # The short, ragged prompts of an ordinary round.
        _prefill("prefill_ragged", groups=32, prompt=(64, 512)),
        # Long prompts, ragged, few of them.
        _prefill("prefill_long", groups=8, prompt=(2048, 4096)),
        # Prompts of a thousand tokens into an fp8 cache.
        _prefill("prefill_fp8", groups=32, prompt=(1024, 1024), dtype="fp8"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["attention", "attention", "append", "projections", "prep", "prefill", "prefill"])
    ratio = rng.choice([1, 2, 2, 4, 8])
    hkv = rng.choice([2, 4, 8, 8])
    d = rng.choice([64, 128, 128])
    dtype = rng.choice(["bf16", "bf16", "fp8"])
    if call == "prefill":
        hi = _log_int(rng, 32, 4096)
        c = _prefill("", hq=hkv * ratio, hkv=hkv, d=d, groups=_log_int(rng, 1, 64), prompt=(rng.randint(1, hi), hi),
                     dtype=dtype)
        while work(c)["flops"] > 4.0e11:
            c["groups"] = max(1, c["groups"] // 2)
    else:
        lo = rng.randint(1, 512)
        hi = _log_int(rng, 32, 32768)
        resp = (float(max(8, hi // 5)), 0.9, hi) if rng.random() < 0.3 else (rng.randint(0, hi // 2), hi)
        group_size = rng.randint(1, 16)
        groups = _log_int(rng, 1, 128)
        live = rng.randint(max(groups, groups * group_size // 2), groups * group_size) if rng.random() < 0.3 else 0
        c = _decode("", call, hq=hkv * ratio, hkv=hkv, d=d, groups=groups, group_size=group_size,
                    prefix=(lo, rng.randint(lo, 1024)), resp=resp, live=live, dtype=dtype,
                    k_mult=rng.choice([0.5, 1.0]))
        # The bytes of a "prep" call do not grow with the lengths, its pool does.
        while _decode_tokens(c) * hkv * d * 4 > 1.2e10:
            c["groups"], c["live"] = max(1, c["groups"] // 2), 0
    del c["name"]
    return c


# ---- sizes ---------------------------------------------------------------------------------------------------------

def _quantiles(lo, hi, n):
    return [int(lo + (hi - lo + 1) * (i + 0.5) / n) for i in range(n)]


def _prefix_lens(c):
    return _quantiles(c["prefix_lo"], c["prefix_hi"], c["groups"])


def _num_seqs(c):
    return c["live"] or c["groups"] * c["group_size"]


def _resp_lens(c):
    """Cached response tokens of every sequence, before the append of a call that has one."""
    n = _num_seqs(c)
    if not c["resp_sigma"]:
        return _quantiles(c["resp_lo"], c["resp_hi"], n)
    z = statistics.NormalDist()
    return [min(c["resp_hi"], int(round(c["resp_lo"] * math.exp(c["resp_sigma"] * z.inv_cdf((i + 0.5) / n)))))
            for i in range(n)]


def _appends(c):
    return c["call"] in ("append", "projections", "prep")


def _decode_tokens(c):
    return sum(_prefix_lens(c)) + sum(_resp_lens(c)) + (_num_seqs(c) if _appends(c) else 0)


def work(case):
    c = case
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    eb = 1 if c["dtype"] == "fp8" else 2
    kv_row = hkv * d * 2 * eb  # one token's K and V in the cache
    scales = 8 * hkv if c["dtype"] == "fp8" else 0  # per page
    if c["call"] == "prefill":
        lens = _prefix_lens(c)
        T = sum(lens)
        byts = T * (hq * d * 2 * 2 + hkv * d * 2 * 2 + hq * 4 + kv_row) + sum(-(-p // PAGE) for p in lens) * scales
        return {"bytes": float(byts), "flops": float(sum(2 * p * (p + 1) * hq * d for p in lens))}
    S = _num_seqs(c)
    qkv_in = S * (hq + 2 * hkv) * d * 2
    if c["call"] == "prep":
        return {"bytes": float(qkv_in + S * (hq * d * 2 + kv_row)), "flops": float(S * (hq + hkv) * d * 8)}
    P, L = _prefix_lens(c), [n + (1 if _appends(c) else 0) for n in _resp_lens(c)]
    pages = sum(-(-n // PAGE) for n in P) + sum(-(-n // PAGE) for n in L)
    byts = (sum(P) + sum(L)) * kv_row + pages * scales + S * (hq * d * 2 * 2 + hq * 4)
    if c["call"] == "append":
        byts += S * (hkv * d * 4 + kv_row)
    if c["call"] == "projections":
        byts += qkv_in + S * (hq * d * 2 + kv_row)
    mean_prefix = sum(P) / len(P)
    return {"bytes": float(byts), "flops": 4.0 * hq * d * (sum(L) + S * mean_prefix)}


# ---- inputs --------------------------------------------------------------------------------------------------------

def _bf16_normal(shape, gen, mult=1.0):
    x = torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    return x.mul_(mult) if mult != 1.0 else x


def _fp8_pool(num_pages, hkv, d, rows_valid, gen, mult):
    """Codes and per-(page, kv-head) scales amax / 448 over each page's valid rows."""
    codes = torch.empty((num_pages, hkv, PAGE, d), dtype=torch.uint8, device="cuda")
    scale = torch.empty((num_pages, hkv), dtype=torch.float32, device="cuda")
    rows = torch.arange(PAGE, device="cuda").view(1, 1, PAGE, 1)
    step = max(1, (1 << 28) // (hkv * PAGE * d))
    for p in range(0, num_pages, step):
        x = torch.empty((min(step, num_pages - p), hkv, PAGE, d), dtype=torch.float32, device="cuda")
        x.normal_(generator=gen).mul_(mult)
        x.mul_(rows < rows_valid[p:p + x.shape[0]].view(-1, 1, 1, 1))
        amax = x.abs().amax(dim=(2, 3))
        s = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
        scale[p:p + x.shape[0]] = s
        codes[p:p + x.shape[0]] = (x / s[:, :, None, None]).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    return codes, scale


def _i32(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda()


def _tables(rng, lens, perm, start):
    """Block table of the given lengths (at least one column) over perm[start:], and the next free entry."""
    pages = [-(-int(n) // PAGE) for n in lens]
    bt = np.zeros((len(pages), max(1, max(pages))), dtype=np.int32)
    for i, n in enumerate(pages):
        bt[i, :n] = perm[start:start + n]
        start += n
    return bt, start


def _layout(c, rng):
    """Lengths, the sequence-to-group map and the block tables of a decode case, on the host."""
    G, S = c["groups"], _num_seqs(c)
    P = np.array(_prefix_lens(c))[rng.permutation(G)]
    L = np.array(_resp_lens(c))[rng.permutation(S)]
    if c["live"]:  # between 1 and group_size live sequences per group, in no particular order
        slots = np.repeat(np.arange(G), c["group_size"] - 1)
        s2g = np.concatenate([np.arange(G), rng.permutation(slots)[:S - G]])
        s2g = s2g[rng.permutation(S)]
    else:
        s2g = np.repeat(np.arange(G), c["group_size"])
    have = L + (1 if _appends(c) else 0)
    num_pages = int((-(-P // PAGE)).sum() + (-(-have // PAGE)).sum())
    perm = rng.permutation(max(1, num_pages))
    pbt, n = _tables(rng, P, perm, 0)
    rbt, n = _tables(rng, have, perm, n)
    rows_valid = np.full(max(1, num_pages), PAGE)
    for bt, lens in ((pbt, P), (rbt, L)):
        for i, n in enumerate(lens):
            if n % PAGE:
                rows_valid[bt[i, n // PAGE]] = n % PAGE
    return P, L, s2g, pbt, rbt, rows_valid


def prepare(case, seed):
    c = case
    rng = np.random.default_rng([seed, 17])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    scale = 1.0 / math.sqrt(d)
    if c["call"] == "prefill":
        P = np.array(_prefix_lens(c))[rng.permutation(c["groups"])]
        offs = np.concatenate([[0], np.cumsum(P)])
        T, num_pages = int(offs[-1]), int((-(-P // PAGE)).sum())
        pbt, _ = _tables(rng, P, rng.permutation(num_pages), 0)
        pool = [torch.zeros((num_pages, hkv, PAGE, d), dtype=torch.uint8 if c["dtype"] == "fp8" else torch.bfloat16,
                            device="cuda") for _ in range(2)]
        sc = [torch.zeros((num_pages, hkv), dtype=torch.float32, device="cuda") for _ in range(2)] \
            if c["dtype"] == "fp8" else [None, None]
        b = rp.PrefillBatch(q=_bf16_normal((T, hq, d), gen), k=_bf16_normal((T, hkv, d), gen),
                            v=_bf16_normal((T, hkv, d), gen), prompt_offs=_i32(offs), prefix_block_table=_i32(pbt),
                            k_pages=pool[0], v_pages=pool[1], k_scale=sc[0], v_scale=sc[1], num_q_heads=hq,
                            softmax_scale=scale)
        return {"case": c, "batch": b, "lens": P.tolist(), "tables": (pbt,)}

    P, L, s2g, pbt, rbt, rows_valid = _layout(c, rng)
    S, num_pages = _num_seqs(c), len(rows_valid)
    ks = vs = None
    if c["dtype"] == "fp8":
        rv = torch.from_numpy(rows_valid).cuda()
        kp, ks = _fp8_pool(num_pages, hkv, d, rv, gen, c["k_mult"])
        vp, vs = _fp8_pool(num_pages, hkv, d, rv, gen, 1.0)
    else:
        kp = _bf16_normal((num_pages, hkv, PAGE, d), gen, c["k_mult"])
        vp = _bf16_normal((num_pages, hkv, PAGE, d), gen)
    new = {}
    if c["call"] == "append":
        new = dict(k_new=_bf16_normal((S, hkv, d), gen, c["k_mult"]), v_new=_bf16_normal((S, hkv, d), gen))
    b = rp.DeviceBatch(k_pages=kp, v_pages=vp, k_scale=ks, v_scale=vs, seq_to_group=_i32(s2g), prefix_lens=_i32(P),
                       prefix_block_table=_i32(pbt), resp_lens=_i32(L), resp_block_table=_i32(rbt),
                       q=_bf16_normal((S, hq, d), gen), num_q_heads=hq, softmax_scale=scale, append=_appends(c), **new)
    if c["call"] in ("projections", "prep"):
        # A few channels dominate, as in trained projections; norm weights around one.
        x = [(_bf16_normal((S, h, d), gen) * torch.exp(0.5 * _bf16_normal((h, d), gen))).contiguous()
             for h in (hq, hkv, hkv)]
        w = [torch.exp(0.3 * _bf16_normal((d,), gen)) for _ in range(2)]
        b.set_projections(*x, *w)
    return {"case": c, "batch": b, "lens": (P.tolist(), L.tolist()), "s2g": s2g.tolist(), "tables": (pbt, rbt)}


def _pool(b):
    return {"k_pages": b.k_pages, "v_pages": b.v_pages, "k_scale": b.k_scale, "v_scale": b.v_scale}


def run(state):
    b, call = state["batch"], state["case"]["call"]
    if call == "prefill":
        b.prefill()
        return {"out": b.out, "lse": b.lse, **_pool(b)}
    if call == "attention":
        b.attention()
        return {"out": b.out, "lse": b.lse}
    if call == "append":
        b.step()
        return {"out": b.out, "lse": b.lse, **_pool(b)}
    if call == "prep":
        b.qk_prep()
        return {"q": b.q, **_pool(b)}
    b.qk_prep_plan()
    b.attn_parts()
    b.combine_parts()
    return {"out": b.out, "lse": b.lse, "q": b.q, **_pool(b)}


def tolerance(case):
    # Outputs are bf16: against 64 bits they are 1.7e-3 off (the rounding of the result, and of the probabilities
    # where they meet a matrix core). fp8 codes are whole values and stay the same.
    return {"rel": 7e-3, "max": 0.1}


# ---- the same in 64 bits -------------------------------------------------------------------------------------------

def _attend(q, k, v, scale, causal=False):
    """q [hq][nq][d], k, v [hkv][n][d], float64 on the GPU: out [hq][nq][d], lse [hq][nq]."""
    hq, nq, d = q.shape
    hkv, n = k.shape[:2]
    out, lse = [], []
    for h in range(hkv):
        s = torch.matmul(q[h * (hq // hkv):(h + 1) * (hq // hkv)].reshape(-1, d), k[h].t().contiguous()) * scale
        s = s.view(-1, nq, n)
        if causal:
            s.masked_fill_(torch.ones((nq, n), dtype=torch.bool, device=s.device).triu_(1), -math.inf)
        e = torch.logsumexp(s, dim=-1)
        lse.append(e)
        out.append(torch.matmul(s.sub_(e[..., None]).exp_().view(-1, n), v[h]).view(-1, nq, d))
    return torch.cat(out), torch.cat(lse)


def _rows(pages, scales, table, n):
    """The first n tokens of a block table, [hkv][n][d] in float64."""
    ids = torch.from_numpy(np.asarray(table[:-(-n // PAGE)], dtype=np.int64)).cuda()
    x = pages[ids]
    x = x.view(torch.float8_e4m3fn).to(torch.float32).double() * scales[ids].double()[:, :, None, None] \
        if scales is not None else x.double()
    return x.transpose(0, 1).reshape(x.shape[1], -1, x.shape[3])[:, :n].contiguous()


def _norm_rotate(x, w, pos, eps, theta):
    """RMS norm and rotary embedding of x [S][h][d] at positions pos [S], float64."""
    d = x.shape[-1]
    x, w = x.double(), w.double()
    y = x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * w
    freq = theta ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=x.device) / d)
    a = (pos.double()[:, None] * freq)[:, None, :]
    lo, hi = y[..., :d // 2], y[..., d // 2:]
    return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], dim=-1)


def exact(case, seed):
    c = case
    st = prepare(c, seed)
    b = st["batch"]
    if c["call"] == "prefill":
        outs, lses, first = [], [], 0
        pool = [torch.zeros_like(b.k_pages), torch.zeros_like(b.v_pages)] if c["dtype"] == "bf16" else [None, None]
        for g, P in enumerate(st["lens"]):
            q, k, v = (x[first:first + P] for x in (b.q, b.k, b.v))
            o, e = _attend(*(x.double().transpose(0, 1).contiguous() for x in (q, k, v)), b.softmax_scale, causal=True)
            outs.append(o.transpose(0, 1))
            lses.append(e.t())
            for pages, x in zip(pool, (k, v)):
                if pages is not None:
                    full = torch.zeros((-(-P // PAGE) * PAGE, c["hkv"], c["d"]), dtype=x.dtype, device="cuda")
                    full[:P] = x
                    ids = torch.from_numpy(st["tables"][0][g, :-(-P // PAGE)].astype(np.int64)).cuda()
                    pages[ids] = full.view(-1, PAGE, c["hkv"], c["d"]).transpose(1, 2)
            first += P
        pool = [x if x is None else x.double() for x in pool]
        return {"out": torch.cat(outs), "lse": torch.cat(lses), "k_pages": pool[0], "v_pages": pool[1],
                "k_scale": None, "v_scale": None}

    P, L = st["lens"]
    pbt, rbt = st["tables"]
    none = {"k_pages": None, "v_pages": None, "k_scale": None, "v_scale": None}
    q, new = b.q.double(), None
    if c["call"] in ("projections", "prep"):
        pos = torch.tensor([P[g] + n for g, n in zip(st["s2g"], L)], device="cuda")
        q = _norm_rotate(b.q_in, b.q_norm_w, pos, b.rms_eps, b.rope_theta)
        if c["call"] == "prep":
            return {"q": q, **none}
        k = _norm_rotate(b.k_in, b.k_norm_w, pos, b.rms_eps, b.rope_theta)
        new = (k.to(torch.bfloat16), b.v_in)
    elif c["call"] == "append":
        new = (b.k_new, b.v_new)
    if new is not None and c["dtype"] == "fp8":
        # The append's scale rule in whole pages: raise the scale where the new row needs it, requantise the rows
        # before it, then store the row.
        at = torch.tensor([rbt[s, n // PAGE] for s, n in enumerate(L)], device="cuda")
        row = torch.tensor([n % PAGE for n in L], device="cuda")
        for pages, scales, x in ((b.k_pages, b.k_scale, new[0]), (b.v_pages, b.v_scale, new[1])):
            amax = x.float().abs().amax(-1)
            old = scales[at]
            fresh = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
            s = torch.where((row == 0)[:, None] | (amax > 448.0 * old), fresh, old)
            vals = pages[at].view(torch.float8_e4m3fn).float() * old[:, :, None, None]
            vals = vals / s[:, :, None, None]
            vals[torch.arange(len(L), device="cuda"), :, row] = x.float() / s[..., None]
            pages[at] = vals.nan_to_num_(0.0).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
            scales[at] = s
    elif new is not None:
        at = torch.tensor([rbt[s, n // PAGE] for s, n in enumerate(L)], device="cuda")
        row = torch.tensor([n % PAGE for n in L], device="cuda")
        b.k_pages[at, :, row] = new[0]
        b.v_pages[at, :, row] = new[1]
    qr = q.to(torch.bfloat16).double()  # the attention reads the q buffer, which is bf16
    outs, lses = [], []
    prefix = {g: (_rows(b.k_pages, b.k_scale, pbt[g], P[g]), _rows(b.v_pages, b.v_scale, pbt[g], P[g]))
              for g in set(st["s2g"])}
    for s, g in enumerate(st["s2g"]):
        n = L[s] + (1 if new is not None else 0)
        k = torch.cat([prefix[g][0], _rows(b.k_pages, b.k_scale, rbt[s], n)], dim=1)
        v = torch.cat([prefix[g][1], _rows(b.v_pages, b.v_scale, rbt[s], n)], dim=1)
        o, e = _attend(qr[s][:, None, :], k, v, b.softmax_scale)
        outs.append(o[:, 0])
        lses.append(e[:, 0])
    r = {"out": torch.stack(outs), "lse": torch.stack(lses)}
    if c["call"] == "projections":
        r["q"] = q
    return {**r, **(none if c["call"] != "attention" else {})}
