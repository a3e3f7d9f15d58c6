"""Measured cases of the compose-and-attend path, called as a serving program calls it.

Each case is one layer's call through the binding of the C ABI, on a plan that the
program has built and uploaded for its batch of requests (a plan is shared by all
layers, so it is in hand before a layer's call):

  fused    c2kv_compose_attend: prefill of a new suffix straight over the stored chunks
  paged    c2kv_compose, then c2kv_attend: prefill that keeps the composed cache
  compose  c2kv_compose alone: the composed cache of a batch is written into pages
  decode   c2kv_attend with one (or a few) new tokens over pages composed beforehand
  sif      c2kv_attend on an extraction plan: originals and compression tokens of a chunk

Keys, values and suffix keys and values are N(0, 1); queries have a standard deviation
of 2, so that attention is peaked rather than nearly uniform.  int8 pools are quantised
per (token, kv-head) from such values.  Everything is drawn from the seed alone.
"""
import math

import numpy as np
import torch

import paper_2607_17715_amd as c2kv

_TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, path, hq, hkv, d, pool, *, batch=1, chunks=1, chunk_len=512, keep_lo=0.25,
          keep_hi=0.25, pattern="random", prefix=0, suffix=1, page=64, base=5e5,
          pre_rope=False, compressed=False, sif_block=0, sif_sink=0):
    c = dict(path=path, hq=hq, hkv=hkv, d=d, pool=pool, batch=batch, chunks=chunks,
             chunk_len=chunk_len, keep_lo=keep_lo, keep_hi=keep_hi, pattern=pattern,
             prefix=prefix, suffix=suffix, page=page, base=base, pre_rope=pre_rope,
             compressed=compressed, sif_block=sif_block, sif_sink=sif_sink)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a small fp32 layer: the smallest prefill, where launches and latency count
        _case("tiny-fp32", "fused", 8, 2, 64, "f32", chunks=4, chunk_len=256, keep_lo=0.5,
              keep_hi=0.5, prefix=16, suffix=32, base=1e4),
        # one Llama-3-8B-shaped layer: a short question over a few retrieved documents
        _case("llama-layer", "fused", 32, 8, 128, "bf16", chunks=8, chunk_len=512, prefix=64,
              suffix=64),
        # a batch of requests with ragged contexts, each over 16 documents
        _case("ragged-batch", "fused", 32, 8, 128, "bf16", batch=16, chunks=16, chunk_len=512,
              keep_lo=0.1, keep_hi=0.5, suffix=128),
        # a long context stored in int8, a short question
        _case("int8-layer", "fused", 32, 8, 128, "i8", chunks=64, chunk_len=1024, keep_lo=0.125,
              keep_hi=0.125, suffix=32),
        # int8 storage, ragged, a longer prompt of odd length, chunks stored compressed
        _case("int8-ragged", "fused", 32, 8, 128, "i8", batch=3, chunks=24, chunk_len=700,
              keep_lo=0.15, keep_hi=0.4, prefix=37, suffix=333, compressed=True),
        # a small model with three query heads per kv-head, keys stored before RoPE and
        # the kept tokens at block ends
        _case("small-prerope", "fused", 12, 4, 64, "bf16", batch=2, chunks=5, chunk_len=601,
              keep_lo=0.125, keep_hi=0.125, pattern="blocks", prefix=13, suffix=45,
              pre_rope=True),
        # 70B-shaped layer, a long prompt over 32k composed tokens, cache kept in pages
        _case("70b-long-suffix", "paged", 64, 8, 128, "bf16", chunks=32, chunk_len=2048,
              keep_lo=0.5, keep_hi=0.5, suffix=2048),
        # the composed cache of an int8 batch written to pages
        _case("compose-int8", "compose", 32, 8, 128, "i8", batch=8, chunks=16, chunk_len=1024,
              keep_lo=0.1, keep_hi=0.5, suffix=16),
        # one decode step over an uncompressed 128k context
        _case("decode-128k", "decode", 32, 8, 128, "bf16", chunks=64, chunk_len=2048, keep_lo=1.0,
              keep_hi=1.0),
        # one decode step over a 16k context compressed 8 times
        _case("decode-16k-8x", "decode", 32, 8, 128, "bf16", chunks=8, chunk_len=2048,
              keep_lo=0.125, keep_hi=0.125),
        # one decode step of a serving batch with ragged contexts
        _case("decode-batch", "decode", 32, 8, 128, "bf16", batch=24, chunks=12, chunk_len=1024,
              keep_lo=0.1, keep_hi=0.5, page=128),
        # extraction: 16 documents of 512 tokens with one compression token per 4
        _case("sif-extract", "sif", 32, 8, 128, "bf16", batch=16, chunk_len=512, sif_block=4,
              sif_sink=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    """Work in units that compare cases: bf16-rate flops, or bytes at 300 flops a byte."""
    w = work(case)
    slow = 16 if case["pool"] == "f32" else 1
    return max(w["flops"] * slow, w["bytes"] * 300)


def draw(rng):
    most = _cost(next(c for c in listed() if c["name"] == "70b-long-suffix"))
    while True:
        path = rng.choice(["fused", "fused", "fused", "paged", "compose", "decode", "decode", "sif"])
        hq, hkv = rng.choice([(32, 8), (32, 8), (64, 8), (16, 4), (8, 2), (12, 4), (8, 8)])
        d = rng.choice([128, 128, 64])
        pool = rng.choice(["bf16", "bf16", "bf16", "i8", "i8", "f32"])
        if path == "sif":
            c = _case(None, path, hq, hkv, d, "f32" if pool == "f32" else "bf16",
                      batch=_log_int(rng, 1, 32), chunk_len=_log_int(rng, 48, 2048),
                      sif_block=rng.choice([4, 8, 10, 16]), sif_sink=rng.choice([0, 4, 16]))
        else:
            suffix = {"fused": (1, 768), "paged": (64, 2048), "compose": (1, 64),
                      "decode": (1, 4)}[path]
            lo = rng.uniform(0.05, 1.0)
            c = _case(None, path, hq, hkv, d, pool, batch=_log_int(rng, 1, 24),
                      chunks=_log_int(rng, 1, 64), chunk_len=_log_int(rng, 64, 2048), keep_lo=lo,
                      keep_hi=min(1.0, lo * rng.uniform(1.0, 3.0)),
                      pattern=rng.choice(["random", "random", "blocks"]),
                      prefix=rng.choice([0, 0, 16, 61]), suffix=_log_int(rng, *suffix),
                      page=rng.choice([64, 64, 128, 256]), base=rng.choice([1e4, 5e5]),
                      pre_rope=rng.random() < 0.2, compressed=rng.random() < 0.3)
        tokens = c["batch"] * (c["prefix"] + c["chunks"] * c["chunk_len"] * c["keep_hi"])
        if _cost(c) <= most and tokens <= 400_000 and c["batch"] * c["suffix"] <= 4096:
            return c


# ---- layout: which tokens are kept, and where they sit in the pool -------------------


def _layout(case, seed):
    """Segments of every request (prefix first, then its chunks) over a pool of distinct
    chunks, with the kept tokens of each."""
    rng = np.random.Generator(np.random.PCG64(seed))
    n, p, b = case["chunk_len"], case["prefix"], case["batch"]
    total = b * case["chunks"] if b * case["chunks"] <= 256 else max(256, case["chunks"])
    kept = []
    for _ in range(total):
        r = rng.uniform(case["keep_lo"], case["keep_hi"])
        if case["pattern"] == "blocks":
            k = max(1, round(1.0 / r))
            kept.append(np.minimum((np.arange(-(-n // k)) + 1) * k, n) - 1)
        else:
            m = min(n, max(1, int(r * n)))
            kept.append(np.sort(rng.choice(n, size=m, replace=False)))
    if case["compressed"]:
        row0 = p + np.concatenate([[0], np.cumsum([len(x) for x in kept])])
        rows = int(row0[-1])
    else:
        row0 = p + n * np.arange(total + 1)
        rows = p + n * total
    seg, req = [], [0]
    for _ in range(b):
        if p:
            seg.append((0, p, np.arange(p)))
        for c in rng.choice(total, size=case["chunks"], replace=False):
            seg.append((int(row0[c]), n, kept[c]))
        req.append(len(seg))
    return dict(rows=rows, req_seg_off=np.array(req, np.int32),
                row0=np.array([s[0] for s in seg], np.int64),
                span=np.array([s[1] for s in seg], np.int32),
                kept=[np.asarray(s[2], np.int32) for s in seg])


def _page_capacity(case):
    m = case["chunk_len"]
    if case["pattern"] != "blocks":
        m = max(1, int(case["keep_hi"] * m))
    return case["batch"] * -(-(case["prefix"] + case["chunks"] * m) // case["page"])


def _normal(gen, shape, dtype, std=1.0):
    return (torch.randn(shape, generator=gen, device="cuda") * std).to(dtype)


def _tensors(case, seed, rows, cached=True):
    """The pool and the new tokens' q, k and v before RoPE, in that order of the seed."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    act = _TORCH["f32" if case["pool"] == "f32" else "bf16"]
    t = {}
    if cached:
        for x in ("k", "v"):
            v = _normal(gen, (rows, case["hkv"], case["d"]), act)
            if case["pool"] == "i8":
                s = v.float().abs().amax(dim=-1) / 127.0
                t[x] = torch.round(v.float() / s[..., None]).clamp_(-127, 127).to(torch.int8)
                t[x + "_scale"] = s.contiguous()
            else:
                t[x] = v
    b, s, d = case["batch"], _new_tokens(case), case["d"]
    t["q"] = _normal(gen, (b, s, case["hq"], d), act, 2.0)
    t["k_suf"] = _normal(gen, (b, s, case["hkv"], d), act)
    t["v_suf"] = _normal(gen, (b, s, case["hkv"], d), act)
    return t


def _new_tokens(case):
    if case["path"] == "sif":
        return case["chunk_len"] + -(-case["chunk_len"] // case["sif_block"])
    return case["suffix"]


def prepare(case, seed):
    act = "f32" if case["pool"] == "f32" else "bf16"
    cached = case["path"] != "sif"
    lay = _layout(case, seed) if cached else None
    t = _tensors(case, seed, lay["rows"] if cached else 0, cached)
    if cached:
        off = np.concatenate([[0], np.cumsum([len(k) for k in lay["kept"]])]).astype(np.int32)
        plan = c2kv.Plan(case["hq"], case["hkv"], case["d"], act, case["base"],
                         lay["req_seg_off"], lay["row0"], lay["span"],
                         np.zeros(len(lay["span"]), np.int32), off, np.concatenate(lay["kept"]),
                         case["suffix"], page_size=case["page"], keys_pre_rope=case["pre_rope"],
                         pool_compressed=case["compressed"])
    else:
        plan = c2kv.Plan.sif(case["hq"], case["hkv"], case["d"], act, case["base"], case["batch"],
                             case["chunk_len"], case["sif_block"], case["sif_sink"])
    plan.upload()
    st = dict(path=case["path"], plan=plan, q=t["q"], k_suf=t["k_suf"], v_suf=t["v_suf"],
              out=torch.empty_like(t["q"]),
              lse=torch.empty((case["batch"], case["hq"], _new_tokens(case)),
                              dtype=torch.float32, device="cuda"))
    if cached:
        st["rows"] = (t["k"], t["v"], t.get("k_scale"), t.get("v_scale"))
        st["pool"] = c2kv.pool_desc(*st["rows"])
    if case["path"] in ("paged", "compose", "decode"):
        # a server's page buffers are of one size, whatever the batch at hand needs of
        # them (zeroed once: nothing writes past a request's last key tile)
        n = _page_capacity(case)
        ks, vs = c2kv.page_shapes(plan)
        st["k_pages"] = torch.zeros((n, *ks[1:]), dtype=_TORCH[act], device="cuda")
        st["v_pages"] = torch.zeros((n, *vs[1:]), dtype=_TORCH[act], device="cuda")
    if case["path"] == "decode":
        # a decode step finds the composed cache of its prefill; the pool is not read again
        c2kv.c2kv_compose(plan, st["pool"], st["k_pages"], st["v_pages"])
        torch.cuda.current_stream().synchronize()
        del st["rows"], st["pool"]
    return st


def run(st):
    path, plan = st["path"], st["plan"]
    if path == "fused":
        c2kv.c2kv_compose_attend(plan, st["pool"], st["q"], st["k_suf"], st["v_suf"], st["out"],
                                 st["lse"])
        return {"out": st["out"], "lse": st["lse"]}
    if path in ("paged", "compose"):
        c2kv.c2kv_compose(plan, st["pool"], st["k_pages"], st["v_pages"])
        if path == "compose":
            return {"k_pages": st["k_pages"], "v_pages": st["v_pages"]}
        c2kv.c2kv_attend(plan, st["k_pages"], st["v_pages"], st["q"], st["k_suf"], st["v_suf"],
                         st["out"], st["lse"])
        return {"out": st["out"], "lse": st["lse"], "k_pages": st["k_pages"],
                "v_pages": st["v_pages"]}
    pages = (st["k_pages"], st["v_pages"]) if path == "decode" else (None, None)
    c2kv.c2kv_attend(plan, *pages, st["q"], st["k_suf"], st["v_suf"], st["out"], st["lse"])
    return {"out": st["out"], "lse": st["lse"]}


# ---- what a pass cannot do without -----------------------------------------------------


def _kept_tokens(case):
    """Composed tokens of the whole batch (the expected number where the kept share is drawn)."""
    n = case["chunk_len"]
    r = 0.5 * (case["keep_lo"] + case["keep_hi"])
    m = -(-n // max(1, round(1.0 / r))) if case["pattern"] == "blocks" else max(1, int(r * n))
    return case["batch"] * (case["prefix"] + case["chunks"] * m)


def work(case):
    hq, hkv, d, b, s = case["hq"], case["hkv"], case["d"], case["batch"], _new_tokens(case)
    act = 4 if case["pool"] == "f32" else 2
    row = 2 * hkv * d                                    # elements of a token's K and V
    new = b * s * ((2 * hq * d + row) * act + 4 * hq)    # q, out, new k and v, lse
    if case["path"] == "sif":
        n, k, sink = case["chunk_len"], case["sif_block"], case["sif_sink"]
        m = -(-n // k)
        pairs = n * (n + 1) // 2 + m * (m + 1) // 2 + m * (k + sink)
        return {"bytes": new, "flops": 4.0 * hq * d * b * pairs}
    kept = _kept_tokens(case)
    pool = kept * (row * {"f32": 4, "bf16": 2, "i8": 1}[case["pool"]] +
                   (8 * hkv if case["pool"] == "i8" else 0))
    flops = 4.0 * hq * d * (kept * s + b * s * (s + 1) // 2)
    pages = kept * row * act
    if case["path"] == "compose":
        return {"bytes": pool + pages, "flops": 3.0 * kept * row}
    if case["path"] == "paged":
        return {"bytes": pool + pages + new, "flops": flops}
    return {"bytes": (pages if case["path"] == "decode" else pool) + new, "flops": flops}


def tolerance(case):
    # fp32: sums in another order (6.6e-7 from 64 bits).  bf16: the scaled query, the
    # turned key, the probabilities and the split partials are each rounded to 8 bits of
    # mantissa (outputs 4e-3 to 6e-3 from 64 bits); a composed page is one rounding of
    # the turned key (1.6e-3).
    if case["pool"] == "f32":
        return {"rel": 4e-6, "max": 2e-4}
    return {"rel": 1.5e-2, "max": 0.2}


# ---- the same in 64 bits, in plain torch ------------------------------------------------


def _rope(x, pos, base):
    """x [tokens, heads, d] turned by pos [tokens], pairs (i, i + d/2)."""
    h = x.shape[-1] // 2
    theta = base ** (-torch.arange(h, dtype=torch.float64, device=x.device) / h)
    ang = pos.to(torch.float64)[:, None, None] * theta
    c, s = torch.cos(ang), torch.sin(ang)
    a, b = x[..., :h], x[..., h:]
    return torch.cat([a * c - b * s, a * s + b * c], dim=-1)


def _attend(q, k, v, visible):
    """q [s, hq, d], k and v [keys, hkv, d]; visible(rows) -> [rows, keys] or None for all."""
    s, hq, d = q.shape
    g = hq // k.shape[1]
    out = torch.empty_like(q)
    lse = torch.empty((hq, s), dtype=torch.float64, device=q.device)
    step = max(1, 100_000_000 // k.shape[0])
    for h in range(hq):
        kt, vh = k[:, h // g].t().contiguous(), v[:, h // g].contiguous()
        for r in range(0, s, step):
            rows = torch.arange(r, min(s, r + step), device=q.device)
            sc = (q[rows, h] @ kt) / math.sqrt(d)
            sc.masked_fill_(~visible(rows), -math.inf)
            z = torch.logsumexp(sc, dim=-1)
            lse[h, rows] = z
            out[rows, h] = torch.exp(sc - z[:, None]) @ vh
    return out, lse


def exact(case, seed):
    dev, f64 = "cuda", torch.float64
    if case["path"] == "sif":
        t = _tensors(case, seed, 0, False)
        n, k, m = case["chunk_len"], case["sif_block"], -(-case["chunk_len"] // case["sif_block"])
        i = torch.arange(n + m, device=dev)
        j = i - n                                        # index of a compression token
        pos = torch.where(i < n, i, torch.clamp((j + 1) * k, max=n) - 1)

        def visible(rows):
            r, u = rows[:, None], i[None]
            own = (u >= (r - n) * k) & (u < (r - n + 1) * k) & (u < n)
            comp = ((u >= n) & (u <= r)) | (u < case["sif_sink"]) | own
            return torch.where(r < n, (u <= r), comp)

        got = [_attend(_rope(t["q"][b].to(f64), pos, case["base"]),
                       _rope(t["k_suf"][b].to(f64), pos, case["base"]), t["v_suf"][b].to(f64),
                       visible) for b in range(case["batch"])]
        return {"out": torch.stack([o for o, _ in got]), "lse": torch.stack([z for _, z in got])}

    lay = _layout(case, seed)
    t = _tensors(case, seed, lay["rows"])
    s, ps, outs, lses, kp, vp = case["suffix"], case["page"], [], [], [], []
    for b in range(case["batch"]):
        rows, new, turn, pos0 = [], [], [], 0
        for c in range(lay["req_seg_off"][b], lay["req_seg_off"][b + 1]):
            kept = lay["kept"][c].astype(np.int64)
            rows.append(lay["row0"][c] + (np.arange(len(kept)) if case["compressed"] else kept))
            turn.append(pos0 + kept if case["pre_rope"] else np.full(len(kept), pos0))
            pos0 += int(lay["span"][c])
        rows = torch.from_numpy(np.concatenate(rows)).to(dev)
        turn = torch.from_numpy(np.concatenate(turn)).to(dev)
        k, v = t["k"][rows].to(f64), t["v"][rows].to(f64)
        if case["pool"] == "i8":
            k *= t["k_scale"][rows].to(f64)[..., None]
            v *= t["v_scale"][rows].to(f64)[..., None]
        k = _rope(k, turn, case["base"])
        n = k.shape[0]
        if case["path"] in ("paged", "compose"):
            np_ = -(-n // ps)
            pad = torch.zeros((np_ * ps - n,) + tuple(k.shape[1:]), dtype=f64, device=dev)
            kp.append(torch.cat([k, pad]).reshape(np_, ps, case["hkv"], -1).permute(0, 2, 1, 3))
            vp.append(torch.cat([v, pad]).reshape(np_, ps, case["hkv"], -1).permute(0, 2, 3, 1))
        if case["path"] != "compose":
            pos = pos0 + torch.arange(s, device=dev)
            u = torch.arange(n + s, device=dev)
            o, z = _attend(_rope(t["q"][b].to(f64), pos, case["base"]),
                           torch.cat([k, _rope(t["k_suf"][b].to(f64), pos, case["base"])]),
                           torch.cat([v, t["v_suf"][b].to(f64)]),
                           lambda r: u[None] <= n + r[:, None])
            outs.append(o)
            lses.append(z)
    got = {}
    if outs:
        got.update(out=torch.stack(outs), lse=torch.stack(lses))
    if kp:
        kp, vp = torch.cat(kp), torch.cat(vp)
        rest = _page_capacity(case) - kp.shape[0]
        got.update(k_pages=torch.cat([kp, kp.new_zeros((rest, *kp.shape[1:]))]),
                   v_pages=torch.cat([vp, vp.new_zeros((rest, *vp.shape[1:]))]))
    return got
