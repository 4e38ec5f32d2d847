"""What a program that serves multi-chunk prompts has this library do, as cases that can be timed and compared.

Every case goes through `paper_2603_05353_amd.Layer`, the library's public binding, on buffers that such a
program keeps from layer to layer.  `op` says which part of the path it is:

  reposition   stage 1: chunk caches -> concatenated, re-rotated caches
  score        stage 2: prompt-conditioned score of every context token
  select       stage 3: the k best tokens
  update       between selection and attention: rotary embedding of the freshly projected query and key rows at
               their global positions, then stage 5 (the new rows replace the cached ones)
  attend       stage 4: causal attention of some rows over the whole cache -- the selected tokens (spread over the
               context) or the prompt's own rows (the last rows of the cache)
  layer        stages 1, 2, 5 and 4 of one small layer, one after the other

Shapes are those of the repository's own configurations (an fp32 layer with 1K tokens of context, 8 heads and
head_dim 64; 32/8 heads of 128 in bf16 at 8K, 32K and about 128K tokens; 28/4 heads at 20K) and, for bf16 layers
with head_dim 64, the 32/8 shape with half the head.  Values are Gaussian with logits of standard deviation one;
a share of the context keys leans towards the prompt, which is what the scoring stage is there to find.
"""
import math

import torch

from paper_2603_05353_amd import Layer

DEV = "cuda:0"
THETA = 5e5
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    wide = dict(dtype="bf16", hq=32, hkv=8, d=128)
    return [
        # the whole path for the smallest layer there is: launches and their gaps, fp32 arithmetic
        dict(name="layer-1k-f32", op="layer", dtype="f32", hq=8, hkv=8, d=64, n=1024, m=32, ratio=0.15, chunks=4, ragged=False),
        # a small bf16 model (heads of 64) on a prompt of uneven documents
        dict(name="layer-8k-d64", op="layer", dtype="bf16", hq=32, hkv=8, d=64, n=8161, m=64, ratio=0.15, chunks=16, ragged=True),
        # assembling a 32K context from 64 cached documents in another order
        dict(name="reposition-32k", op="reposition", n=32768, chunks=64, ragged=False, pairing="half", **wide),
        # scoring it with a prompt of 128 tokens
        dict(name="score-32k-m128", op="score", n=32768, m=128, prompt_keys=False, **wide),
        # an 8K context whose scores are normalised as a real forward pass would, prompt keys included
        dict(name="score-8k-prompt-keys", op="score", n=8192, m=64, prompt_keys=True, **wide),
        # choosing 15 % of 32K and 10 % of a long, odd-sized context
        dict(name="select-32k", op="select", n=32768, ratio=0.15, spread=0.002),
        dict(name="select-130k", op="select", n=130078, ratio=0.10, spread=0.3),
        # bringing the recomputed rows of a 32K context into the cache
        dict(name="update-32k", op="update", n=32768, ratio=0.15, pairing="half", **wide),
        # attention of the selected rows: 32K, the grouped heads of a vision-language layer at 20K, and 130K tokens
        dict(name="attend-32k", op="attend", n=32768, ratio=0.15, rows=0, lse=False, **wide),
        dict(name="attend-20k-g7", op="attend", dtype="bf16", hq=28, hkv=4, d=128, n=20480, ratio=0.15, rows=0, lse=False),
        dict(name="attend-130k", op="attend", n=130078, ratio=0.10, rows=0, lse=False, **wide),
        # the prompt's own 128 rows over the finished 32K cache, the last step before decoding
        dict(name="attend-prompt-32k", op="attend", n=32768 + 128, ratio=0.0, rows=128, lse=True, **wide),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes spread over the logarithm of the range, most of them odd."""
    hq, hkv = rng.choice([(32, 8), (32, 8), (28, 4), (40, 8), (16, 16), (16, 2), (64, 8)])
    shape = dict(dtype="bf16", hq=hq, hkv=hkv, d=128)
    op = rng.choice(["reposition", "score", "score", "select", "update", "attend", "attend", "attend", "layer", "layer"])
    n = _log_int(rng, 1000, 131072)
    if op == "reposition":
        return dict(op=op, n=n, chunks=max(1, min(96, n // rng.choice([128, 256, 512, 1024]))), ragged=rng.random() < 0.7,
                    pairing=rng.choice(["half", "half", "interleaved"]), **shape)
    if op == "score":
        return dict(op=op, n=n, m=_log_int(rng, 4, 256), prompt_keys=rng.random() < 0.4, **shape)
    if op == "select":
        return dict(op=op, n=n, ratio=round(rng.uniform(0.01, 0.4), 3), spread=rng.choice([0.002, 0.05, 0.3, 1.0]))
    if op == "update":
        return dict(op=op, n=n, ratio=round(rng.uniform(0.02, 0.3), 3), pairing=rng.choice(["half", "half", "interleaved"]), **shape)
    if op == "attend":
        if rng.random() < 0.35:
            rows = _log_int(rng, 1, 256)
            return dict(op=op, n=n + rows, ratio=0.0, rows=rows, lse=rng.random() < 0.5, **shape)
        ratio = rng.uniform(0.03, 0.3)
        ratio = min(ratio, 1.2e13 / (2.0 * 128 * hq * n * n))       # no more work than the largest listed case
        return dict(op=op, n=n, ratio=round(ratio, 4), rows=0, lse=rng.random() < 0.3, **shape)
    # small layers on the other types: fp32, and heads of 64
    dtype, d = rng.choice([("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 64), ("bf16", 128)])
    hq, hkv = rng.choice([(8, 8), (16, 4), (32, 8), (14, 2)])
    n = _log_int(rng, 200, 1600 if dtype == "f32" else 8000)
    return dict(op="layer", dtype=dtype, hq=hq, hkv=hkv, d=d, n=n, m=_log_int(rng, 4, 64), ratio=round(rng.uniform(0.05, 0.2), 3),
                chunks=max(1, min(32, n // 200)), ragged=rng.random() < 0.7)


# ---------------------------------------------------------------------------------------------------------------
# Inputs.  Everything is made on the GPU from the seed; the CPU generator only decides chunk lengths and their order.
# ---------------------------------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _chunk_plan(case, seed):
    """Lengths of the chunks (they add up to n) and their order in the concatenation."""
    g = torch.Generator().manual_seed(int(seed) + 17)
    n, c = case["n"], case["chunks"]
    if case["ragged"]:
        w = torch.rand(c, generator=g, dtype=torch.float64) + 0.25
        cuts = torch.cumsum(w, 0) / w.sum() * n
        ends = [int(x) for x in cuts.tolist()]
        ends[-1] = n
        lens = [b - a for a, b in zip([0] + ends[:-1], ends)]
    else:
        lens = [n // c] * c
        lens[-1] += n - sum(lens)
    return lens, torch.randperm(c, generator=g).tolist()


def _rows_at(case, seed):
    """Positions of the rows that are recomputed, ascending: a random `ratio` of the context, or its last rows."""
    n = case["n"]
    if case.get("rows"):
        return torch.arange(n - case["rows"], n, dtype=torch.int32, device=DEV)
    k = max(1, math.floor(case["ratio"] * n))
    return torch.sort(torch.randperm(n, generator=_gen(seed + 5), device=DEV)[:k])[0].to(torch.int32)


def _inputs(case, seed):
    """The case's tensors, before any of the library's work."""
    op, g = case["op"], _gen(seed)
    x = {}
    if op == "select":
        n = case["n"]
        s = torch.exp(case["spread"] * torch.randn(n, generator=g, device=DEV))
        lean = torch.rand(n, generator=g, device=DEV) < 0.05
        x["scores"] = torch.where(lean, s * (1.0 + 3.0 * case["spread"]), s) * (128.0 / n)
        return x
    dt = DTYPES[case["dtype"]]
    n, hq, hkv, d = case["n"], case["hq"], case["hkv"], case["d"]

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=DEV)

    # a direction per kv head that prompt queries share and some keys lean towards
    lean = normal(hkv, d)
    lean /= lean.norm(dim=-1, keepdim=True)
    if op in ("score", "layer"):
        m = case["m"]
        x["q_prompt"] = (normal(m, hq, d) + 2.0 * lean.repeat_interleave(hq // hkv, 0)).to(dt)
    keys = normal(n, hkv, d)
    if op != "reposition":
        keys += 4.0 * lean * (torch.rand(n, 1, 1, generator=g, device=DEV) < 0.05)
    x["k"] = keys.to(dt)
    del keys
    if op != "score":
        x["v"] = normal(n, hkv, d).to(dt)
    if op == "score" and case["prompt_keys"]:
        x["k_prompt"] = normal(case["m"], hkv, d).to(dt)
    if op in ("update", "attend", "layer"):
        x["pos"] = _rows_at(case, seed)
        r = x["pos"].numel()
        x["q"] = normal(r, hq, d).to(dt)
        if op != "attend":
            x["k_new"], x["v_new"] = normal(r, hkv, d).to(dt), normal(r, hkv, d).to(dt)
    return x


def prepare(case, seed):
    op, x = case["op"], _inputs(case, seed)
    s = dict(x, op=op, case=case)
    if op == "select":
        s["layer"] = Layer("bf16", 32, 8, 128, THETA, max_ctx=case["n"], max_prompt=1)
        s["idx"] = torch.empty(max(1, s["layer"].budget_of(case["n"], case["ratio"])), dtype=torch.int32, device=DEV)
        return s
    L = s["layer"] = Layer(case["dtype"], case["hq"], case["hkv"], case["d"], THETA, max_ctx=case["n"],
                           max_prompt=case.get("m", 1), pairing=case.get("pairing", "half"))
    if op in ("reposition", "layer"):
        lens, s["order"] = _chunk_plan(case, seed)
        # each document's cache is an allocation of its own
        s["k_chunks"] = [t.clone() for t in torch.split(x["k"], lens)]
        s["v_chunks"] = [t.clone() for t in torch.split(x["v"], lens)]
        s["k_out"], s["v_out"] = L.empty_cache(case["n"]), L.empty_cache(case["n"])
        del s["k"], s["v"]
    if op in ("score", "layer"):
        s["scores"] = torch.empty(case["n"], dtype=torch.float32, device=DEV)
    if op in ("attend", "layer"):
        s["out"] = torch.empty_like(x["q"])
    if op == "reposition":  # a call with dozens of chunk pointers is marshalled once and repeated
        s["call"] = L.bind("reposition_keys", s["k_chunks"], s["v_chunks"], chunk_order=s["order"], k_out=s["k_out"],
                           v_out=s["v_out"])
    return s


def run(s):
    op, L, case = s["op"], s["layer"], s["case"]
    if op == "select":
        return {"idx": L.select_topk(s["scores"], ratio=case["ratio"], idx_out=s["idx"])}
    if op == "reposition":
        s["call"]()
        return {"k": s["k_out"], "v": s["v_out"]}
    if op == "score":
        return {"scores": L.score_tokens(s["k"], s["q_prompt"], k_prompt=s.get("k_prompt"), scores=s["scores"])}
    if op == "update":
        L.rope_rows(s["q"], s["pos"])
        L.rope_rows(s["k_new"], s["pos"])
        L.splice_kv(s["k_new"], s["v_new"], s["pos"], s["k"], s["v"])
        return {"q": s["q"], "k": s["k"], "v": s["v"]}
    if op == "attend":
        if case["lse"]:
            out, lse = L.recompute_attention(s["q"], s["pos"], s["k"], s["v"], out=s["out"], return_lse=True)
            return {"out": out, "lse": lse}
        return {"out": L.recompute_attention(s["q"], s["pos"], s["k"], s["v"], out=s["out"])}
    L.reposition_score(s["k_chunks"], s["v_chunks"], s["q_prompt"], chunk_order=s["order"], k_out=s["k_out"],
                       v_out=s["v_out"], scores=s["scores"])
    L.splice_kv(s["k_new"], s["v_new"], s["pos"], s["k_out"], s["v_out"])
    L.recompute_attention(s["q"], s["pos"], s["k_out"], s["v_out"], out=s["out"])
    return {"k": s["k_out"], "v": s["v_out"], "scores": s["scores"], "out": s["out"]}


# ---------------------------------------------------------------------------------------------------------------
# What a pass cannot do without.
# ---------------------------------------------------------------------------------------------------------------
def work(case):
    op, n = case["op"], case["n"]
    if op == "select":
        return {"bytes": 4.0 * n + 4.0 * math.floor(case["ratio"] * n), "flops": 0.0}
    e = 2 if case["dtype"] == "bf16" else 4
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    row, qrow = hkv * d * e, hq * d * e
    k = case.get("rows") or max(1, math.floor(case.get("ratio", 0) * n))
    # causal keys of k rows spread over the context, or of its last k rows
    keys = k * (n - (k - 1) / 2.0) if case.get("rows") else k * (n + 1) / 2.0
    b = f = 0.0
    if op in ("reposition", "layer"):
        b += 4.0 * n * row
    if op in ("score", "layer"):
        m = case["m"]
        b += n * row + m * qrow + 4.0 * n + (m * row if case.get("prompt_keys") else 0)
        # one product; a second one only because the normaliser of a row is known after all its keys
        f += 2 * 2.0 * n * m * hq * d
        f += 2.0 * hq * d * m * (m + 1) / 2 if case.get("prompt_keys") else 0
    if op == "update":
        b += 2.0 * k * (qrow + row)          # rotary embedding, in place
    if op in ("update", "layer"):
        b += 4.0 * k * row + 4.0 * k         # splice
    if op in ("attend", "layer"):
        b += 2.0 * n * row + 2.0 * k * qrow + 4.0 * k
        f += 4.0 * d * hq * keys
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times what two correct evaluations differ by, measured against `exact` rounded to the storage type."""
    op = case["op"]
    if op == "select":
        return "exact"
    if op == "attend":      # bf16 probabilities and one bf16 rounding of the result
        return {"rel": 1e-2}
    if op == "score":       # fp32 logits, exponentials and sums
        return {"rel": 1e-5}
    if op == "layer":
        return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}
    return {"rel": 2e-4}    # fp32 rotation, rounded once: now and then to the other neighbour


# ---------------------------------------------------------------------------------------------------------------
# The same results in 64 bits, from the definitions.
# ---------------------------------------------------------------------------------------------------------------
def _rotate(x, pos, pairing):
    """Rotary embedding of x [T, H, d] (float64) at positions pos [T]."""
    d = x.shape[-1]
    freq = THETA ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device=DEV) / d)
    ang = pos.to(torch.float64)[:, None] * freq[None, :]
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    out = torch.empty_like(x)
    if pairing == "half":
        a, b = x[..., : d // 2], x[..., d // 2:]
        out[..., : d // 2], out[..., d // 2:] = a * c - b * s, a * s + b * c
    else:
        a, b = x[..., 0::2], x[..., 1::2]
        out[..., 0::2], out[..., 1::2] = a * c - b * s, a * s + b * c
    return out


def _assemble(case, x, seed):
    lens, order = _chunk_plan(case, seed)
    ks, vs = torch.split(x["k"], lens), torch.split(x["v"], lens)
    k, v, at = [], [], 0
    for c in order:
        k.append(_rotate(ks[c].double(), torch.full((lens[c],), at, device=DEV), case.get("pairing", "half")))
        v.append(vs[c].double())
        at += lens[c]
    return torch.cat(k), torch.cat(v)


def _score(case, k, x):
    m, hq, hkv, d = case["m"], case["hq"], case["hkv"], case["d"]
    n, grp, scale = k.shape[0], hq // hkv, d ** -0.5
    total = torch.zeros(n, dtype=torch.float64, device=DEV)
    for h in range(hq):
        kh = k[:, h // grp, :].double().contiguous()
        q = x["q_prompt"][:, h, :].double().contiguous()
        logits = torch.mm(q, kh.t().contiguous()) * scale
        z = torch.logsumexp(logits, 1)
        if case.get("prompt_keys"):
            kp = x["k_prompt"][:, h // grp, :].double().contiguous()
            lp = torch.mm(q, kp.t().contiguous()) * scale
            lp = lp.masked_fill(torch.ones(m, m, dtype=torch.bool, device=DEV).triu(1), -math.inf)
            z = torch.logaddexp(z, torch.logsumexp(lp, 1))
        total += torch.exp(logits - z[:, None]).sum(0)
    return total / hq


def _attend(case, q, pos, k, v):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    r, grp, scale = q.shape[0], hq // hkv, d ** -0.5
    out = torch.empty(r, hq, d, dtype=torch.float64, device=DEV)
    lse = torch.empty(r, hq, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 28) // (k.shape[0] * grp))     # at most 2 GiB of logits at a time
    for g in range(hkv):
        kt, vg = k[:, g, :].double().t().contiguous(), v[:, g, :].double().contiguous()
        for r0 in range(0, r, step):
            p = pos[r0:r0 + step].long()
            top = int(p[-1]) + 1
            qs = q[r0:r0 + step, g * grp:(g + 1) * grp, :].double().reshape(-1, d).contiguous()
            logits = torch.mm(qs, kt[:, :top].contiguous()).mul_(scale).view(p.numel(), grp, top)
            logits.masked_fill_((torch.arange(top, device=DEV)[None, :] > p[:, None])[:, None, :], -math.inf)
            ls = torch.logsumexp(logits, 2)
            w = logits.sub_(ls[..., None]).exp_()
            o = torch.mm(w.view(-1, top), vg[:top].contiguous())
            out[r0:r0 + step, g * grp:(g + 1) * grp, :] = o.view(p.numel(), grp, d)
            lse[r0:r0 + step, g * grp:(g + 1) * grp] = ls
    return out, lse


def exact(case, seed):
    op, x = case["op"], _inputs(case, seed)
    if op == "select":
        s = x["scores"].double()
        k = math.floor(case["ratio"] * case["n"])
        return {"idx": torch.sort(torch.sort(s, descending=True, stable=True)[1][:k])[0].to(torch.int32)}
    if op == "reposition":
        k, v = _assemble(case, x, seed)
        return {"k": k, "v": v}
    if op == "score":
        return {"scores": _score(case, x["k"], x)}
    if op == "attend":
        out, lse = _attend(case, x["q"], x["pos"], x["k"], x["v"])
        return {"out": out, "lse": lse} if case["lse"] else {"out": out}
    if op == "update":
        k, v, pos = x["k"].double(), x["v"].double(), x["pos"].long()
        k[pos] = _rotate(x["k_new"].double(), pos, case["pairing"])
        v[pos] = x["v_new"].double()
        return {"q": _rotate(x["q"].double(), pos, case["pairing"]), "k": k, "v": v}
    # a layer: the caches hold their storage type between the stages
    k, v = _assemble(case, x, seed)
    pos, stored = x["pos"].long(), k.to(DTYPES[case["dtype"]]).double()
    scores = _score(case, stored, x)
    for t in (k, stored):
        t[pos] = x["k_new"].double()
    v[pos] = x["v_new"].double()
    out, _ = _attend(case, x["q"], x["pos"], stored, v)
    return {"k": k, "v": v, "scores": scores, "out": out}
