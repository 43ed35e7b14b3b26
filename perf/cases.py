"""The work users have this library do, as measurable cases.

Each case is one call of a public entry point (the step classes of
``paper_2609_03311_amd.pipeline`` and ``dopr_store_put``) on the shapes of the
repository's own workloads: Qwen3-0.6B-, 4B- and 8B-shaped layers and a
Llama-3.2-1B-shaped one, prefix budgets of 8 to 512 slots, 1 to 129 online
tokens per pair, from one query's candidates to a batch of 64 queries,
salience selection of 64- to 2048-token documents, and store ingest.

The integer structure of a case (token counts, prefix lengths, which pairs
share a document) follows from the case alone; a seed relabels the documents,
reorders the pairs and draws every value.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2609_03311_amd import dopr_store_create, dopr_store_put, pipeline
from paper_2609_03311_amd import dopr_store_bytes

DEV = "cuda"
EPS = 1e-6
THETA = 1e6
TOP_P = 8
RATIO = 8

# (q heads, kv heads, head size, QK-norm) of the models' attention layers
SHAPES = {
    "0p6b": (16, 8, 128, True),
    "8b": (32, 8, 128, True),         # the 4B layer has the same heads
    "llama8b": (32, 8, 128, False),
    "llama1b": (32, 8, 64, False),
}
# (hidden, intermediate) of the whole decoder layers
WIDTHS = {"0p6b": (1024, 3072), "4b": (2560, 9728), "8b": (4096, 12288)}


def _attn(name, shape, pairs, docs, slots, toks, reuse, ids=0, kind="attn",
          width="", layout=0):
    return {"name": name, "kind": kind, "shape": shape, "pairs": pairs,
            "docs": docs, "ids": ids or docs, "slots_lo": slots[0],
            "slots_hi": slots[1], "tok_lo": toks[0], "tok_hi": toks[1],
            "reuse": reuse, "width": width, "layout": layout}


def _salience(name, shape, docs, lens, layout=0):
    return {"name": name, "kind": "salience", "shape": shape, "docs": docs,
            "len_lo": lens[0], "len_hi": lens[1], "layout": layout}


def listed():
    return [
        # four short queries against eight documents: the latency of a call
        _attn("attn_tiny", "0p6b", 32, 8, (16, 16), (16, 16), "queries"),
        # one query reranked against its 100 candidates, 2048-token
        # documents at 8x: the smallest request a server answers
        _attn("attn_8b_one_query", "8b", 100, 1000, (256, 256), (129, 129),
              "queries"),
        # a batch of 64 short queries x 100 passages of 256 tokens
        _attn("attn_0p6b", "0p6b", 6400, 10000, (32, 32), (32, 32),
              "queries"),
        # Zipf-popular documents of 512 tokens, queries of 8 to 64 tokens
        _attn("attn_4b_zipf", "8b", 4096, 20000, (64, 64), (9, 65), "zipf"),
        # the large uniform batch: 64 long queries x 100 long documents
        _attn("attn_8b", "8b", 6400, 5000, (256, 256), (129, 129),
              "queries"),
        # everything ragged, a million document ids of which only the
        # batch's are resident, half of the pairs on popular documents
        _attn("attn_8b_ragged", "8b", 4096, 0, (8, 256), (17, 129), "half",
              ids=1_000_000),
        # the other model family: head size 64, no QK-norm, given rotary
        # frequencies
        _attn("attn_llama1b", "llama1b", 6400, 5000, (256, 256), (129, 129),
              "queries"),
        # last-layer scoring of the large batch
        _attn("score_8b", "8b", 6400, 5000, (256, 256), (129, 129),
              "queries", kind="score"),
        # a whole decoder layer, 16 queries x 100 passages
        _attn("layer_0p6b", "0p6b", 1600, 2500, (32, 32), (32, 32),
              "queries", kind="layer", width="0p6b"),
        # offline: which slots of 16 long documents are kept
        _salience("salience_8b", "8b", 16, (2048, 2048)),
        # offline: 512 passages
        _salience("salience_0p6b", "0p6b", 512, (256, 256)),
        # offline: the kept slots of 4,000 documents enter the store
        {"name": "ingest_8b", "kind": "ingest", "shape": "8b", "docs": 4000,
         "slots_lo": 256, "slots_hi": 256, "layout": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["attn", "score", "layer", "salience", "ingest"],
                       [45, 20, 10, 15, 10])[0]
    layout = rng.randrange(1 << 30)
    if kind == "salience":
        shape = rng.choice(["0p6b", "8b"])
        hi = _log_int(rng, 64, 2048)
        lo = hi if rng.random() < 0.4 else max(1, int(hi * rng.uniform(.2, 1)))
        hq = SHAPES[shape][0]
        most = 32 * 16 * 2048 ** 2 // (hq * hi * hi)
        docs = _log_int(rng, 1, max(1, min(512, most)))
        c = _salience("", shape, docs, (lo, hi), layout)
        del c["name"]
        return c
    hi = _log_int(rng, 8, 512)
    lo = hi if rng.random() < 0.4 else max(1, int(hi * rng.uniform(0.05, 1)))
    if kind == "ingest":
        shape = rng.choice(["0p6b", "llama1b"])
        docs = _log_int(rng, 8, max(8, min(20000, 4000 * 256 // hi)))
        return {"kind": kind, "shape": shape, "docs": docs, "slots_lo": lo,
                "slots_hi": hi, "layout": layout}
    t_hi = _log_int(rng, 8, 129)
    t_lo = t_hi if rng.random() < 0.4 else max(1, int(t_hi * rng.uniform(0.1,
                                                                         1)))
    if kind == "layer":
        width = rng.choice(["0p6b", "4b", "8b"])
        shape = "0p6b" if width == "0p6b" else "8b"
        most = {"0p6b": 51200, "4b": 8000, "8b": 4000}[width] // t_hi
    else:
        width = ""
        shape = rng.choice(["0p6b", "8b", "8b", "llama8b", "llama1b"])
        # no more keys seen in all than by the large batch's rows
        most = min(6400, 6400 * 129 * 321 // (t_hi * (hi + t_hi // 2 + 1)))
    pairs = _log_int(rng, 8, max(8, most))
    reuse = rng.choice(["queries", "queries", "zipf", "half"])
    # no more resident slots than the large batch's store
    docs = max(8, min(int(pairs * rng.uniform(0.3, 3)), 5000 * 256 // hi))
    ids = docs
    if reuse == "half":
        docs, ids = 0, rng.choice([2 * pairs, 100_000, 1_000_000])
    c = _attn("", shape, pairs, docs, (lo, hi), (t_lo, t_hi), reuse, ids=ids,
              kind=kind, width=width, layout=layout)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Integer structure

def _zipf(rng, n, count):
    w = np.arange(1, n + 1, dtype=np.float64) ** -1.1
    cdf = np.cumsum(w)
    ranks = np.searchsorted(cdf / cdf[-1], rng.random(count), side="right")
    return rng.permutation(n)[np.minimum(ranks, n - 1)]


def _structure(case):
    """(doc_len [ids] with -1 = not resident, doc_ids [P], tokens [P])."""
    rng = np.random.default_rng(case["layout"])
    n, P = case["ids"], case["pairs"]
    doc_len = rng.integers(case["slots_lo"], case["slots_hi"] + 1, n)
    toks = rng.integers(case["tok_lo"], case["tok_hi"] + 1, P)
    if case["reuse"] == "queries":
        per = min(100, n)
        ids = np.concatenate([rng.choice(n, per, replace=False)
                              for _ in range(-(-P // per))])[:P]
    elif case["reuse"] == "zipf":
        ids = _zipf(rng, n, P)
    else:
        pop = _zipf(rng, n, P // 2)
        rest = np.setdiff1d(np.arange(n), pop)
        ids = np.concatenate([pop, rng.choice(rest, P - P // 2,
                                              replace=False)])
        ids = ids[rng.permutation(P)]
        used = np.zeros(n, bool)
        used[ids] = True
        doc_len = np.where(used, doc_len, -1)
    return (doc_len.astype(np.int32), ids.astype(np.int32),
            toks.astype(np.int32))


def _relabelled(case, seed):
    """The structure under the seed's document names and pair order."""
    doc_len, ids, toks = _structure(case)
    rng = np.random.default_rng([seed, case["layout"]])
    name = rng.permutation(len(doc_len))
    order = rng.permutation(len(ids))
    new_len = np.empty_like(doc_len)
    new_len[name] = doc_len
    return new_len, name[ids][order].astype(np.int32), toks[order]


def _doc_lens(case, lo, hi):
    rng = np.random.default_rng(case["layout"])
    return rng.integers(case[lo], case[hi] + 1, case["docs"]).astype(np.int32)


# ---------------------------------------------------------------------------
# Values

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _randn(g, *shape, scale=1.0, offset=0.0):
    n = math.prod(shape)
    out = torch.empty(n, dtype=torch.bfloat16, device=DEV)
    for a in range(0, n, 1 << 28):
        b = min(n, a + (1 << 28))
        x = torch.randn(b - a, generator=g, device=DEV)
        out[a:b] = x.mul_(scale).add_(offset)
    return out.view(*shape)


def _inv_freq(d):
    """Llama 3's rescaled rotary frequencies."""
    f = 500000.0 ** (-torch.arange(0, d, 2, dtype=torch.float64) / d)
    wave = 2 * math.pi / f
    smooth = ((8192 / wave - 1) / 3).clamp(0, 1)
    return ((1 - smooth) * f / 32 + smooth * f).float().to(DEV)


def _batch(case, seed):
    doc_len, ids, toks = _relabelled(case, seed)
    hq, hkv, d, norm = SHAPES[case["shape"]]
    g = _gen(seed)
    slots = int(doc_len[doc_len >= 0].sum())
    ntok = int(toks.sum())
    b = {"doc_len": doc_len, "doc_ids_h": ids, "toks": toks,
         "k_src": _randn(g, slots, hkv, d), "v_src": _randn(g, slots, hkv, d),
         "doc_ids": torch.from_numpy(ids).to(DEV),
         "cu": torch.from_numpy(np.concatenate(
             [[0], np.cumsum(toks)]).astype(np.int32)).to(DEV)}
    if case["kind"] == "layer":
        w, i = WIDTHS[case["width"]]
        b["x"] = _randn(g, ntok, w)
        b["weights"] = {
            "attn_norm_w": _randn(g, w, scale=0.1, offset=1.0),
            "w_q": _randn(g, hq * d, w, scale=w ** -0.5),
            "w_k": _randn(g, hkv * d, w, scale=w ** -0.5),
            "w_v": _randn(g, hkv * d, w, scale=w ** -0.5),
            "w_o": _randn(g, w, hq * d, scale=(hq * d) ** -0.5),
            "mlp_norm_w": _randn(g, w, scale=0.1, offset=1.0),
            "w_gate": _randn(g, i, w, scale=w ** -0.5),
            "w_up": _randn(g, i, w, scale=w ** -0.5),
            "w_down": _randn(g, w, i, scale=i ** -0.5)}
    else:
        b["q"] = _randn(g, ntok, hq, d)
        b["k"] = _randn(g, ntok, hkv, d)
        b["v"] = _randn(g, ntok, hkv, d)
        b["norm_w"] = _randn(g, hq * d, scale=0.1, offset=1.0)
        b["w_head"] = _randn(g, 2, hq * d, scale=(hq * d) ** -0.5)
    b["qw"] = _randn(g, d, scale=0.1, offset=1.0) if norm else None
    b["kw"] = _randn(g, d, scale=0.1, offset=1.0) if norm else None
    b["kw_rope"] = {} if norm else {"rope_inv_freq": _inv_freq(d)}
    return b


def _slots(case, seed):
    """Source slots of the documents that enter a store, in a seeded order."""
    lens = _doc_lens(case, "slots_lo", "slots_hi")
    hq, hkv, d, _ = SHAPES[case["shape"]]
    rng = np.random.default_rng([seed, case["layout"]])
    lens = lens[rng.permutation(len(lens))]
    ids = rng.permutation(len(lens))
    cu = np.concatenate([[0], np.cumsum(lens[ids].astype(np.int64))])
    g = _gen(seed)
    n = int(lens.sum())
    return (lens, torch.from_numpy(ids.astype(np.int32)).to(DEV),
            torch.from_numpy(cu.astype(np.int64)).to(DEV),
            _randn(g, n, hkv, d), _randn(g, n, hkv, d))


def _docs(case, seed):
    lens = _doc_lens(case, "len_lo", "len_hi")
    lens = lens[np.random.default_rng([seed, case["layout"]])
                .permutation(len(lens))]
    hq, hkv, d, _ = SHAPES[case["shape"]]
    g = _gen(seed)
    n = int(lens.sum())
    return lens, _randn(g, n, hq, d), _randn(g, n, hkv, d)


# ---------------------------------------------------------------------------
# Preparation and one pass

def prepare(case, seed):
    hq, hkv, d, _ = SHAPES[case["shape"]]
    if case["kind"] == "salience":
        lens, q, k = _docs(case, seed)
        step = pipeline.SalienceStep(lens, n_q_heads=hq, n_kv_heads=hkv,
                                     top_p=TOP_P, ratio=RATIO)
        return {"kind": "salience", "step": step, "q": q, "k": k}
    if case["kind"] == "ingest":
        lens, ids, cu, k, v = _slots(case, seed)
        pool_bytes, _ = dopr_store_bytes(1, hkv, d, lens)
        pool = torch.zeros(pool_bytes, dtype=torch.uint8, device=DEV)
        store = dopr_store_create(1, hkv, d, lens, pool=pool)
        return {"kind": "ingest", "store": store, "ids": ids, "cu": cu,
                "k": k, "v": v}
    b = _batch(case, seed)
    store = pipeline.make_store(b["doc_len"], hkv, b.pop("k_src"),
                                b.pop("v_src"))
    shape = {"n_pairs": case["pairs"], "n_q_heads": hq,
             "total_tokens": int(b["toks"].sum()),
             "max_tokens": int(b["toks"].max())}
    if case["kind"] == "attn":
        step = pipeline.OnlineStep(store, **shape)
    elif case["kind"] == "score":
        step = pipeline.ScoreStep(store, **shape)
    else:
        w, i = WIDTHS[case["width"]]
        step = pipeline.LayerStep(store, b["weights"], hidden=w,
                                  intermediate=i, **shape)
    return {"kind": case["kind"], "step": step, **b}


def run(s):
    if s["kind"] == "salience":
        s["step"].run(s["q"], s["k"])
        return [s["step"].u, s["step"].selected]
    if s["kind"] == "ingest":
        dopr_store_put(s["store"], 0, s["ids"], s["cu"], s["k"], s["v"])
        return [s["store"].pool]
    step = s["step"]
    if s["kind"] == "layer":
        step.run(0, s["doc_ids"], s["cu"], s["x"], s["qw"], s["kw"])
        return [step.y]
    if s["kind"] == "attn":
        step.attention(0, s["doc_ids"], s["cu"], s["q"], s["k"], s["v"],
                       s["qw"], s["kw"], **s["kw_rope"])
        step.score_head(s["cu"], s["norm_w"], s["w_head"])
        return [step.out, step.score, step.logits]
    step.run(0, s["doc_ids"], s["cu"], s["q"], s["k"], s["v"], s["qw"],
             s["kw"], s["norm_w"], s["w_head"], **s["kw_rope"])
    return [step.out, step.lse, step.score, step.logits]


# ---------------------------------------------------------------------------
# What a pass cannot do without

def work(case):
    hq, hkv, d, _ = SHAPES[case["shape"]]
    if case["kind"] == "salience":
        n = _doc_lens(case, "len_lo", "len_hi").astype(np.int64)
        tok = int(n.sum())
        # every visible logit of every head once
        return {"bytes": tok * (hq + hkv) * d * 2 + tok * 4
                + int((n // RATIO).sum()) * 4,
                "flops": int((n * (n + 1)).sum()) * hq * d}
    if case["kind"] == "ingest":
        n = int(_doc_lens(case, "slots_lo", "slots_hi").sum())
        return {"bytes": 2 * n * hkv * d * 2 * 2, "flops": 0}
    doc_len, ids, toks = _structure(case)
    T, L = toks.astype(np.int64), doc_len[ids].astype(np.int64)
    ntok, P = int(T.sum()), case["pairs"]
    prefix = int(doc_len[np.unique(ids)].astype(np.int64).sum()) * hkv * d * 4
    own = ntok * hkv * d * 2 * 2
    if case["kind"] == "score":
        return {"bytes": prefix + own + 2 * P * hq * d * 2 + P * hq * 4
                + P * 12, "flops": 4 * hq * d * int((L + T).sum())}
    flops = 4 * hq * d * int((T * L + T * (T + 1) // 2).sum())
    if case["kind"] == "attn":
        return {"bytes": prefix + own + 2 * ntok * hq * d * 2 + P * 12,
                "flops": flops}
    w, i = WIDTHS[case["width"]]
    mats = w * (2 * hq + 2 * hkv) * d + 3 * w * i
    return {"bytes": prefix + 2 * ntok * w * 2 + mats * 2,
            "flops": flops + 2 * ntok * mats}


def tolerance(case):
    # about four times the distance from `exact` measured on the listed and
    # drawn cases: 2.7e-3 to 3.7e-3 for bf16 outputs (2.7e-3 is what q^, the
    # weights and the rows rounded to bf16 give), 5.5e-7 for the salience;
    # a kept position may change where two saliences tie
    if case["kind"] == "ingest":
        return "exact"
    if case["kind"] == "salience":
        return {"rel": 4e-6, "differ": 0.02}
    return {"rel": 1.5e-2}


# ---------------------------------------------------------------------------
# The same in 64 bits

def _rms(x, w):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + EPS) * w


def _rope(x, pos, freq):
    """x [B, T, H, D] rotated at pos [B, T]."""
    a = pos[..., None].double() * freq
    c, s = a.cos()[:, :, None], a.sin()[:, :, None]
    h = x.shape[-1] // 2
    x0, x1 = x[..., :h], x[..., h:]
    return torch.cat([x0 * c - x1 * s, x1 * c + x0 * s], -1)


def _attention64(b, shape, q, k, v, last):
    """Attention rows [Ntok, Hq, D] and log-sum-exp [Ntok, Hq] in float64
    (`last`: of each pair's last token only, [P, ...])."""
    hq, hkv, d, norm = shape
    rep = hq // hkv
    doc_len, ids, toks = b["doc_len"], b["doc_ids_h"], b["toks"]
    freq = (b["kw_rope"]["rope_inv_freq"].double() if not norm else
            THETA ** (-torch.arange(0, d, 2, dtype=torch.float64,
                                    device=DEV) / d))
    start = np.concatenate([[0], np.cumsum(np.maximum(doc_len, 0)
                                           .astype(np.int64))])
    cu = np.concatenate([[0], np.cumsum(toks.astype(np.int64))])
    n_out = len(ids) if last else int(cu[-1])
    out = torch.empty(n_out, hq, d, dtype=torch.float64, device=DEV)
    lse = torch.empty(n_out, hq, dtype=torch.float64, device=DEV)
    L_of = doc_len[ids]
    order = np.lexsort((L_of, toks))
    i = 0
    while i < len(order):
        # pairs of similar size, padded to the batch's largest
        n = 1
        while i + n < len(order):
            sel = order[i:i + n + 1]
            t, m = int(toks[sel].max()), int(L_of[sel].max())
            rows = 1 if last else t
            if (n + 1) * (hq * rows * (m + t) + 4 * hkv * d * (m + t)) > 2**28:
                break
            n += 1
        sel = order[i:i + n]
        i += n
        T, m = int(toks[sel].max()), int(L_of[sel].max())
        tt = torch.from_numpy(toks[sel].astype(np.int64)).to(DEV)
        ll = torch.from_numpy(L_of[sel].astype(np.int64)).to(DEV)
        j = torch.arange(T, device=DEV)
        tok = (torch.from_numpy(cu[sel]).to(DEV)[:, None]
               + torch.minimum(j, tt[:, None] - 1))
        pos = ll[:, None] + j
        kk, vv = k[tok].double(), v[tok].double()
        if norm:
            kk = _rms(kk, b["kw"].double())
        kk = _rope(kk, pos, freq)
        if last:
            qt, qpos = tok[:, -1:], (ll + tt - 1)[:, None]
        else:
            qt, qpos = tok, pos
        qq = q[qt].double()
        if norm:
            qq = _rms(qq, b["qw"].double())
        qq = _rope(qq, qpos, freq)
        s = torch.arange(m, device=DEV)
        if m:
            slot = (torch.from_numpy(start[ids[sel]]).to(DEV)[:, None]
                    + torch.minimum(s, (ll[:, None] - 1).clamp(min=0)))
            kk = torch.cat([b["k_src"][slot].double(), kk], 1)
            vv = torch.cat([b["v_src"][slot].double(), vv], 1)
        B, R = qq.shape[0], qq.shape[1]
        # [B*hkv, R*rep, d] x [B*hkv, d, m+T]
        qa = (qq.view(B, R, hkv, rep, d).permute(0, 2, 1, 3, 4)
              .reshape(B * hkv, R * rep, d))
        ka = kk.permute(0, 2, 3, 1).reshape(B * hkv, d, m + T).contiguous()
        va = vv.permute(0, 2, 1, 3).reshape(B * hkv, m + T, d).contiguous()
        x = torch.bmm(qa, ka).mul_(d ** -0.5).view(B, hkv, R, rep, m + T)
        see = torch.empty(B, R, m + T, dtype=torch.bool, device=DEV)
        see[:, :, :m] = (s < ll[:, None])[:, None]
        qj = qpos - ll[:, None]
        see[:, :, m:] = j <= qj[:, :, None]
        x.masked_fill_(~see[:, None, :, None], -math.inf)
        z = torch.logsumexp(x, -1)
        x = torch.exp_(x.sub_(z[..., None]))
        o = torch.bmm(x.view(B * hkv, R * rep, m + T), va)
        o = (o.view(B, hkv, R, rep, d).permute(0, 2, 1, 3, 4)
             .reshape(B, R, hq, d))
        z = z.permute(0, 2, 1, 3).reshape(B, R, hq)
        if last:
            row = torch.from_numpy(sel).to(DEV)
            out[row], lse[row] = o[:, 0], z[:, 0]
        else:
            ok = j < tt[:, None]
            out[tok[ok]], lse[tok[ok]] = o[ok], z[ok]
    return out, lse


def _head64(h, b):
    y = _rms(h, b["norm_w"].double()) @ b["w_head"].double().t()
    return y[:, 0] - y[:, 1], y


def exact(case, seed):
    hq, hkv, d, _ = shape = SHAPES[case["shape"]]
    if case["kind"] == "ingest":
        return None
    if case["kind"] == "salience":
        return _salience64(case, seed)
    b = _batch(case, seed)
    if case["kind"] == "layer":
        w = {k: v.double() for k, v in b["weights"].items()}
        x = b["x"].double()
        h = _rms(x, w["attn_norm_w"])
        q, k, v = (h @ w[n].t() for n in ("w_q", "w_k", "w_v"))
        a, _ = _attention64(b, shape, q.view(-1, hq, d), k.view(-1, hkv, d),
                            v.view(-1, hkv, d), False)
        x = x + a.view(len(x), hq * d) @ w["w_o"].t()
        h = _rms(x, w["mlp_norm_w"])
        act = torch.nn.functional.silu(h @ w["w_gate"].t()) * (
            h @ w["w_up"].t())
        return [x + act @ w["w_down"].t()]
    last = case["kind"] == "score"
    out, lse = _attention64(b, shape, b["q"], b["k"], b["v"], last)
    h = out if last else out[(b["cu"][1:] - 1).long()]
    s, y = _head64(h.reshape(len(h), hq * d), b)
    return [out, lse, s, y] if last else [out, s, y]


def _salience64(case, seed):
    hq, hkv, d, _ = SHAPES[case["shape"]]
    lens, q, k = _docs(case, seed)
    us, sel, t0 = [], [], 0
    for n in lens.tolist():
        qd = q[t0:t0 + n].double().permute(1, 0, 2)
        kd = k[t0:t0 + n].double().permute(1, 2, 0)
        t0 += n
        mean = torch.zeros(n, n, dtype=torch.float64, device=DEV)
        above = torch.ones(n, n, dtype=torch.bool, device=DEV).triu(1)
        for h in range(hq):
            x = (qd[h] @ kd[h * hkv // hq].contiguous()).mul_(d ** -0.5)
            mean += torch.softmax(x.masked_fill_(above, -math.inf), -1)
        mean /= hq
        # the m = min(p, n - i) largest of column i's visible rows
        m = torch.clamp(n - torch.arange(n, device=DEV), max=TOP_P)
        top = mean.masked_fill(above, -1).topk(min(TOP_P, n), 0).values
        live = torch.arange(len(top), device=DEV)[:, None] < m
        u = torch.where(live, top, 0.).sum(0) / m
        us.append(u)
        best = torch.sort(u, descending=True, stable=True).indices
        sel.append(best[:n // RATIO].sort().values.int())
    return [torch.cat(us), torch.cat(sel)]
