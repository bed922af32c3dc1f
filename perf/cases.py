"""Measured cases of the composed-prefill path: one attention layer of a batch
of requests, or one of its steps, called through a Session as a serving
program calls it.

A case is a batch layout and a step:

  step      "layer"     assemble (compose + append), attention, retain
            "attn"      attention alone over an assembled request KV
            "assemble"  compose + append alone
  kv        "bf16", "e4m3" (bf16 activations) or "f32"
  hq, hkv, d            query heads, KV heads, head dim
  page                  tokens per KV page
  requests              requests in the batch
  units_lo .. units_hi  context units per request, uniform
  len_lo .. len_hi      tokens per unit, uniform, in multiples of len_mult
  miss                  units per request computed from text (the others are
                        cached); below zero: each unit is with probability
                        -miss
  window                leading tokens recomputed of each reused unit
  head, tail            text tokens before and after the units
  scope                 keys that computed units see: "global" or "local"
  alias                 V (and K) of whole cached pages read from the pool:
                        "", "v" or "vk"
  layout                seed of the layout (lengths, units, page order)

The layout follows from the case; the values follow from the seed.
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

from paper_2609_32999_amd import _binding as B
from paper_2609_32999_amd.session import Session

_L8B = dict(hq=32, hkv=8, d=128, page=16, alias="", scope="global")
_DT = {"f32": torch.float32, "bf16": torch.bfloat16, "e4m3": torch.uint8}
_ITEM = {"f32": 4, "bf16": 2, "e4m3": 1}


def listed():
    return [
        # the fp32 reference configuration (4 heads of 64, two of four units
        # of 64 tokens cached): the smallest call, launches and latency
        dict(name="tiny_f32_layer", step="layer", kv="f32", hq=4, hkv=4, d=64, page=16,
             requests=1, units_lo=4, units_hi=4, len_lo=64, len_hi=64, len_mult=1, miss=2,
             window=4, head=0, tail=16, scope="global", alias="", layout=0),
        # a few short agent turns: ragged units at unaligned offsets
        dict(name="short_layer", step="layer", kv="bf16", **_L8B, requests=3, units_lo=3,
             units_hi=6, len_lo=20, len_hi=150, len_mult=1, miss=-0.4, window=5, head=37,
             tail=19, layout=11),
        # one RAG request on its own, 3 of 10 chunks missing: time to first
        # token of an unloaded server
        dict(name="rag_one_layer", step="layer", kv="bf16", **_L8B, requests=1, units_lo=10,
             units_hi=10, len_lo=512, len_hi=512, len_mult=1, miss=3, window=16, head=64,
             tail=32, layout=1),
        # the same with every chunk cached: only windows and text are computed
        dict(name="rag_one_cached_layer", step="layer", kv="bf16", **_L8B, requests=1,
             units_lo=10, units_hi=10, len_lo=512, len_hi=512, len_mult=1, miss=0, window=16,
             head=64, tail=32, layout=2),
        # one RAG request over an fp8 pool
        dict(name="rag_one_fp8_layer", step="layer", kv="e4m3", **_L8B, requests=1,
             units_lo=16, units_hi=16, len_lo=512, len_hi=512, len_mult=16, miss=3, window=16,
             head=64, tail=32, layout=3),
        # the headline RAG batch: its attention, missing chunks over the whole
        # prompt, and with each missing chunk prefilled on its own
        dict(name="rag_attn", step="attn", kv="bf16", **_L8B, requests=8, units_lo=10,
             units_hi=10, len_lo=512, len_hi=512, len_mult=1, miss=3, window=16, head=64,
             tail=32, layout=4),
        dict(name="rag_local_attn", step="attn", kv="bf16", **{**_L8B, "scope": "local"},
             requests=8, units_lo=10, units_hi=10, len_lo=512, len_hi=512, len_mult=1, miss=3,
             window=16, head=64, tail=32, layout=4),
        # agent memory: many short ragged records at unaligned offsets
        dict(name="agent_attn", step="attn", kv="bf16", **_L8B, requests=16, units_lo=20,
             units_hi=60, len_lo=64, len_hi=256, len_mult=1, miss=-0.25, window=8, head=256,
             tail=64, layout=5),
        # long context at 64 query heads (the largest case)
        dict(name="long_attn", step="attn", kv="bf16", **{**_L8B, "hq": 64}, requests=4,
             units_lo=32, units_hi=32, len_lo=1024, len_hi=1024, len_mult=1, miss=3, window=32,
             head=64, tail=32, layout=6),
        # the fp8 pool's batch: attention
        dict(name="fp8_attn", step="attn", kv="e4m3", **_L8B, requests=16, units_lo=16,
             units_hi=16, len_lo=512, len_hi=512, len_mult=16, miss=3, window=16, head=64,
             tail=32, layout=7),
        # placing cached pages and computed rows: the headline batch and the
        # fp8 one
        dict(name="rag_assemble", step="assemble", kv="bf16", **_L8B, requests=8, units_lo=10,
             units_hi=10, len_lo=512, len_hi=512, len_mult=1, miss=3, window=16, head=64,
             tail=32, layout=4),
        dict(name="fp8_assemble", step="assemble", kv="e4m3", **_L8B, requests=16, units_lo=16,
             units_hi=16, len_lo=512, len_hi=512, len_mult=16, miss=3, window=16, head=64,
             tail=32, layout=7),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges, at most the largest listed one's work."""
    while True:
        kv = rng.choice(["bf16", "bf16", "bf16", "e4m3", "e4m3", "f32"])
        c = dict(step=rng.choice(["layer", "attn", "attn", "assemble"]), kv=kv, d=128, page=16,
                 scope=rng.choice(["global", "global", "local"]), alias="",
                 layout=rng.randrange(1 << 20))
        if kv == "f32":
            c["d"] = rng.choice([64, 128])
            g, c["hkv"] = rng.choice([(1, 4), (4, 2), (2, 4)])
            c.update(requests=rng.randint(1, 2), units_lo=2, units_hi=rng.randint(2, 5))
            top = 120
        else:
            g, c["hkv"] = rng.choice([(4, 8), (4, 8), (8, 8), (8, 4), (2, 8), (1, 8)])
            c["requests"] = _log_int(rng, 1, 32)
            c["units_hi"] = _log_int(rng, 3, 48)
            c["units_lo"] = rng.randint(max(1, c["units_hi"] // 3), c["units_hi"])
            top = 1024
        c["hq"] = g * c["hkv"]
        c["len_hi"] = _log_int(rng, 32, top)
        c["len_lo"] = rng.randint(max(16, c["len_hi"] // 4), c["len_hi"])
        c["len_mult"] = 1
        c["miss"] = rng.choice([0, 1, 3, -0.25, -0.4])
        c["window"] = rng.choice([1, 5, 8, 16, 32])
        c["head"] = rng.randint(0, 256)
        c["tail"] = rng.randint(1, 96)
        if kv == "bf16":
            c["page"] = rng.choice([16, 16, 32])
            if c["step"] != "assemble":
                c["alias"] = rng.choice(["", "", "", "", "v", "vk"])
        if kv == "e4m3":
            # page-aligned segments and windows
            c.update(len_mult=16, window=rng.choice([16, 32]), head=16 * rng.randint(0, 16))
        w, costliest = work(c), work(listed()[8])
        if w["flops"] <= costliest["flops"] and w["bytes"] <= costliest["bytes"]:
            return c


# ------------------------------------------------------------------ layout
def _layout(case):
    """Requests of the case, arena sizes and token counts."""
    rng = random.Random(case["layout"])
    mult, page = case["len_mult"], case["page"]
    specs, uid, pool, pages = [], 0, 0, 0
    for _ in range(case["requests"]):
        n = rng.randint(case["units_lo"], case["units_hi"])
        if case["miss"] >= 0:
            missing = set(rng.sample(range(n), min(n, int(case["miss"]))))
        else:
            missing = {i for i in range(n) if rng.random() < -case["miss"]}
        pos = case["head"]
        text = [(0, pos)] if pos else []
        units = []
        for i in range(n):
            ln = max(mult, rng.randint(case["len_lo"], case["len_hi"]) // mult * mult)
            npg = -(-ln // page)
            units.append(SimpleNamespace(
                unit_id=uid, n_tokens=ln, position=pos, residency=int(i not in missing),
                n_recompute=case["window"], retain=int(i in missing), pool_pages=(pool, npg)))
            uid, pool, pos = uid + 1, pool + npg, pos + ln
        text.append((pos, case["tail"]))
        pos += case["tail"]
        npg = -(-pos // page)
        specs.append(SimpleNamespace(prompt_len=pos, units=units, text_segs=text,
                                     block_table=(pages, npg),
                                     miss_scope=int(case["scope"] == "local")))
        pages += npg
    return specs, pool, pages


def _place(case, specs, pool, pages):
    """Non-adjacent pages: both arenas in a random order."""
    rng = np.random.default_rng(case["layout"])
    po, ro = rng.permutation(pool).astype(np.int32), rng.permutation(pages).astype(np.int32)
    for r in specs:
        a, n = r.block_table
        r.block_table = ro[a:a + n]
        for u in r.units:
            a, n = u.pool_pages
            u.pool_pages = po[a:a + n]
    return specs


def _rows(case, spec):
    """Computed positions of a request and the first key each sees."""
    pos, lo = [], []
    segs = [(s, n, None) for s, n in spec.text_segs]
    segs += [(u.position, u.n_tokens, u) for u in spec.units]
    for start, n, u in sorted(segs, key=lambda s: s[0]):
        take = n if u is None or not u.residency else min(n, case["window"])
        p = np.arange(start, start + take)
        first = np.zeros_like(p)
        if u is not None and not u.residency and case["scope"] == "local":
            first[min(n, case["window"]):] = start
        pos.append(p)
        lo.append(first)
    return np.concatenate(pos), np.concatenate(lo)


def work(case):
    specs, _, _ = _layout(case)
    hq, hkv, d, kvb = case["hq"], case["hkv"], case["d"], _ITEM[case["kv"]]
    act = 4 if case["kv"] == "f32" else 2
    T = prompt = gathered = retained = pairs = 0
    for s in specs:
        pos, lo = _rows(case, s)
        T += len(pos)
        prompt += s.prompt_len
        pairs += int((pos + 1 - lo).sum())
        gathered += s.prompt_len - len(pos)
        retained += sum(u.n_tokens for u in s.units if not u.residency)
    token = 2 * hkv * d * kvb                       # K and V of a token
    fresh = 2 * hkv * d * act
    nbytes = flops = 0
    if case["step"] in ("layer", "assemble"):
        nbytes += gathered * 2 * token + T * (fresh + token)
    if case["step"] in ("layer", "attn"):
        nbytes += 2 * T * hq * d * act + T * hq * 4 + prompt * token
        flops += 4 * d * hq * pairs
    if case["step"] == "layer":
        nbytes += retained * (fresh + token)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Pages are copies, or fp32 rotations rounded once in a stated order, and
    # come out the same to the bit.  The error of attention outputs against
    # 64 bits is 1.7e-3 at bf16 (its own rounding, and that of rotated
    # queries and probabilities); another order of its sums moves the
    # roundings of the outputs by under 1e-3.  At fp32 it is 3e-8, one
    # rounding of the output.
    if case["step"] == "assemble":
        return "exact"
    return {"rel": 2e-7} if case["kv"] == "f32" else {"rel": 4e-3}


# ------------------------------------------------------------------ inputs
def _codes(shape, gen):
    """e4m3 codes of N(0, 1) values at page scales 2^-7 .. 2^-5, one element
    of each page at the largest magnitude, as the quantizer leaves them."""
    pages = shape[0]
    scale = torch.exp2(torch.randint(-7, -4, (pages,), generator=gen, device="cuda").float())
    codes = torch.empty(shape, dtype=torch.uint8, device="cuda")
    for a in range(0, pages, 4096):
        x = torch.randn((min(4096, pages - a), *shape[1:]), generator=gen, device="cuda")
        x /= scale[a:a + 4096, None, None, None]
        x[:, 0, 0, 0] = 448.0
        codes[a:a + 4096] = x.clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    return codes, scale


def prepare(case, seed):
    specs, pool, pages = _layout(case)
    _place(case, specs, pool, pages)
    top = max(s.prompt_len for s in specs)
    act = "f32" if case["kv"] == "f32" else "bf16"
    shape = SimpleNamespace(
        n_q_heads=case["hq"], n_kv_heads=case["hkv"], head_dim=case["d"],
        page_size=case["page"], kv_dtype=case["kv"], act_dtype=act,
        rope_theta=10000.0 if act == "f32" else 500000.0, max_position=-(-top // 4096) * 4096)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    sess = Session(shape, pool, pages)
    plan = sess.plan(specs, alias_v="v" in case["alias"], alias_k="k" in case["alias"])
    T = plan.num_compute_tokens
    # cached states, and what an earlier batch left in the request pages
    if case["kv"] == "e4m3":
        for i, arena in enumerate((sess.pool_k, sess.pool_v)):
            arena[0], sess.pool_scale[0, :, i] = _codes(arena.shape[1:], gen)
        for arena in (sess.req_k, sess.req_v, sess.req_scale):
            arena.zero_()
    else:
        for arena in (sess.pool_k, sess.pool_v):
            arena.normal_(generator=gen)
        sess.req_k.zero_()
        sess.req_v.zero_()
    dt = _DT[act]
    q = torch.randn((T, case["hq"], case["d"]), generator=gen, device="cuda").to(dt)
    k = torch.randn((T, case["hkv"], case["d"]), generator=gen, device="cuda").to(dt)
    v = torch.randn((T, case["hkv"], case["d"]), generator=gen, device="cuda").to(dt)
    out, lse = sess.new_outputs(plan)
    out.zero_()
    lse.zero_()
    st = SimpleNamespace(case=case, specs=specs, sess=sess, plan=plan, q=q, k=k, v=v, out=out,
                         lse=lse)
    if case["step"] == "attn":
        sess.assemble(plan, k, v)
    return st


def run(st):
    s, step = st.sess, st.case["step"]
    got = {}
    if step != "attn":
        s.assemble(st.plan, st.k, st.v)
        got.update(req_k=s.req_k, req_v=s.req_v)
        if s.e4m3:
            got.update(req_scale=s.req_scale)
    if step != "assemble":
        s.attn(st.plan, st.q, st.out, st.lse)
        got.update(out=st.out, lse=st.lse)
    if step == "layer":
        s.retain(st.plan, st.k, st.v)
        got.update(pool_k=s.pool_k, pool_v=s.pool_v)
        if s.e4m3:
            got.update(pool_scale=s.pool_scale)
    return got


# --------------------------------------------------------------- reference
def _rotate(x, pos, d, theta):
    """x [n][H][d] rotated in 64 bits at pos [n], pairs (i, i + d/2)."""
    i = torch.arange(d // 2, dtype=torch.float64, device="cuda")
    a = pos.double()[:, None] * (theta ** (-2.0 * i / d))[None]
    c, s = a.cos()[:, None], a.sin()[:, None]
    lo, hi = x[..., : d // 2], x[..., d // 2:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)


def _e4m3(x, dims):
    """x rounded to e4m3 at the smallest power-of-two scale that covers it."""
    amax = x.abs().amax(dims, keepdim=True)
    sc = torch.exp2(torch.ceil(torch.log2(amax / 448.0)))
    sc = torch.where(amax > 0, sc, torch.ones_like(sc))
    return (x / sc).float().to(torch.float8_e4m3fn).double() * sc


def exact(case, seed):
    st = prepare(case, seed)
    s, d, page, hkv = st.sess, case["d"], case["page"], case["hkv"]
    theta = 10000.0 if case["kv"] == "f32" else 500000.0
    g = case["hq"] // hkv
    e4m3 = case["kv"] == "e4m3"

    def tokens(arena, scale, pages, n):
        x = arena[0][torch.as_tensor(pages.astype(np.int64), device="cuda")]
        if e4m3:
            x = x.view(torch.float8_e4m3fn).double()
            x = x * scale[torch.as_tensor(pages.astype(np.int64), device="cuda")].double()[
                :, None, None, None]
        return x.double().permute(0, 2, 1, 3).reshape(-1, hkv, d)[:n]

    def as_stored(x):
        """Computed K or V as an e4m3 page holds it (page-aligned runs)."""
        if not e4m3:
            return x
        return torch.cat([_e4m3(x[a:a + 16], (0, 1, 2)) for a in range(0, len(x), 16)])

    if case["step"] != "assemble":
        out = torch.zeros(st.out.shape, dtype=torch.float64, device="cuda")
        lse = torch.zeros(st.lse.shape, dtype=torch.float64, device="cuda")
    keep = not e4m3 and not case["alias"]
    if keep:
        rk = torch.zeros(s.req_k.shape, dtype=torch.float64, device="cuda")
        rv = torch.zeros(s.req_v.shape, dtype=torch.float64, device="cuda")
    row = 0
    for r in st.specs:
        pos, first = _rows(case, r)
        n = len(pos)
        P = torch.as_tensor(pos, device="cuda")
        lo = torch.as_tensor(first, device="cuda")
        K = torch.zeros((r.prompt_len, hkv, d), dtype=torch.float64, device="cuda")
        V = torch.zeros_like(K)
        for u in r.units:
            w = min(case["window"], u.n_tokens)
            if u.residency and w < u.n_tokens:
                at = torch.arange(u.position + w, u.position + u.n_tokens, device="cuda")
                ps = s.pool_scale[0] if e4m3 else None
                k = tokens(s.pool_k, ps[:, 0] if e4m3 else None, u.pool_pages, u.n_tokens)[w:]
                K[at] = as_stored(_rotate(k, at, d, theta))
                V[at] = tokens(s.pool_v, ps[:, 1] if e4m3 else None, u.pool_pages,
                               u.n_tokens)[w:]
        kr = _rotate(st.k[row:row + n].double(), P, d, theta)
        vr = st.v[row:row + n].double()
        # runs of computed positions that follow one another share pages
        cuts = [0, *(np.nonzero(np.diff(pos) != 1)[0] + 1).tolist(), n]
        K[P] = torch.cat([as_stored(kr[a:b]) for a, b in zip(cuts, cuts[1:])])
        V[P] = torch.cat([as_stored(vr[a:b]) for a, b in zip(cuts, cuts[1:])])
        if keep:
            bt = torch.as_tensor(r.block_table.astype(np.int64), device="cuda")
            at = torch.arange(r.prompt_len, device="cuda")
            for arena, x in ((rk, K), (rv, V)):
                arena[0, bt[at // page], :, at % page] = x
        if case["step"] != "assemble":
            if case["kv"] == "bf16":
                K, V = K.bfloat16().double(), V.bfloat16().double()
            Q = _rotate(st.q[row:row + n].double(), P, d, theta)
            if e4m3:
                Q = _e4m3(Q, (2,))
            for a in range(0, n, 2048):
                b = min(n, a + 2048)
                top = int(pos[a:b].max()) + 1
                at = torch.arange(top, device="cuda")
                hide = (at[None] > P[a:b, None]) | (at[None] < lo[a:b, None])
                for h in range(case["hq"]):
                    S = Q[a:b, h] @ K[:top, h // g].T.contiguous() / math.sqrt(d)
                    S.masked_fill_(hide, -math.inf)
                    m = S.amax(1, keepdim=True)
                    S.sub_(m).exp_()
                    l = S.sum(1, keepdim=True)
                    out[row + a:row + b, h] = (S @ V[:top, h // g]) / l
                    lse[row + a:row + b, h] = (m + l.log())[:, 0]
        row += n
    got = {}
    if case["step"] != "attn":
        got.update(req_k=rk if keep else None, req_v=rv if keep else None)
    if case["step"] != "assemble":
        got.update(out=out, lse=lse)
    return got if any(x is not None for x in got.values()) else None
