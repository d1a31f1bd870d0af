"""The work that a serving stack has this library do, as cases that can be timed and compared.

A check layer scores its reused tokens and picks some (`score`), later layers project, write back and attend with
the picked ones (`attn`, `project`, `chain`); a decode step re-checks every running request (`check`), writes back
and attends with what it picked (`recompute`); the retriever matches a new request's tokens against an earlier one
(`match`); check layers that weight or study the ranking need the attention column mass (`colsum`) and the first-order
impact (`impact`); `tiny` is the whole path on the small fp32 layer.  Shapes are those of `synth.WORKLOADS`, values and
distributions those of `synth`.

Every case goes through `paper_2503_16525_amd.binding`, with buffers and workspaces that the caller keeps.  A pass
leaves its state as it found it, apart from its outputs: a cache that a pass writes to gets the same rows each time.
"""
import math
import random

import torch

from paper_2503_16525_amd import binding as kvs
from paper_2503_16525_amd import synth

DEV = "cuda"
MODELS = {"qwen": synth.QWEN, "llama": synth.LLAMA, "yi": synth.YI, "tiny": synth.TINY}
HASH_BASE, HASH_MODULUS = 1000003, 4294967291


def listed():
    return [
        # the smallest calls: every step of the path on the fp32 layer, where launches and latency are all there is
        dict(name="tiny-layer-f32", kind="tiny", n=512, ratio=0.15),
        # one request of ordinary, odd length: picked in the check layer, recomputed in a later one
        dict(name="chain-qwen-6001", kind="chain", model="qwen", n=6001, ratio=0.10, hidden=3584),
        # a long prompt's check layer
        dict(name="score-llama-32k", kind="score", model="llama", n=32768, ratio=0.15, alpha=False, mode="v"),
        # its picked tokens' attention in each layer
        dict(name="attn-llama-32k", kind="attn", model="llama", n=32768, ratio=0.15),
        # the largest: a context whose K and V outgrow the last-level cache
        dict(name="attn-yi-131k", kind="attn", model="yi", n=131072, ratio=0.10),
        # the projection of what one decode check of a 32k context picks (2 %)
        dict(name="project-llama-656", kind="project", model="llama", n=32768, n_sel=656, hidden=4096, rope=True),
        # the decode check of one long request
        dict(name="check-llama-32k", kind="check", model="llama", batch=1, lo=32768, hi=32768, attn_out=False),
        # and of a full, ragged batch
        dict(name="check-llama-64x", kind="check", model="llama", batch=64, lo=4096, hi=16384, attn_out=False),
        # the write-back and attention of what that batch picks
        dict(name="recompute-llama-64x", kind="recompute", model="llama", batch=64, lo=4096, hi=16384, ratio=0.02),
        # the attention column mass of a check layer
        dict(name="colsum-qwen-8k", kind="colsum", model="qwen", n=8192),
        # the retriever: a prompt against an earlier one
        dict(name="match-32k", kind="match", n=32768, window=16),
        # the first-order impact that the ranking is compared with
        dict(name="impact-qwen-8k", kind="impact", model="qwen", n=8192),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["tiny", "chain", "score", "attn", "project", "check", "check", "recompute", "colsum", "match", "impact"])
    model = rng.choice(["qwen", "llama", "yi"])
    ratio = round(rng.uniform(0.05, 0.30), 3)
    hidden = rng.choice([1024, 2048, 3584, 4096])
    if kind == "tiny":
        return dict(kind=kind, n=_log(rng, 64, 2048), ratio=ratio)
    if kind == "chain":
        return dict(kind=kind, model=model, n=_log(rng, 1024, 32768), ratio=ratio, hidden=hidden)
    if kind == "score":
        return dict(kind=kind, model=model, n=_log(rng, 1024, 131072), ratio=ratio, alpha=rng.random() < 0.5, mode=rng.choice(["v", "v", "kv"]))
    if kind == "attn":
        # from a decode check's 2 % to a prefill's 30 %, and no more work than the largest listed case
        n = _log(rng, 1024, 131072)
        most = 1.3e13 / (4 * 128 * MODELS[model].n_q_heads * 0.5 * n * n)
        return dict(kind=kind, model=model, n=n, ratio=round(min(math.exp(rng.uniform(math.log(0.02), math.log(0.30))), most), 4))
    if kind == "project":
        return dict(kind=kind, model=model, n=32768, n_sel=_log(rng, 1, 9000), hidden=hidden, rope=rng.random() < 0.75)
    if kind == "check":
        if rng.random() < 0.4:
            n = _log(rng, 1024, 131072)
            return dict(kind=kind, model=model, batch=1, lo=n, hi=n, attn_out=rng.random() < 0.25)
        hi = _log(rng, 1024, 16384)
        return dict(kind=kind, model=model, batch=_log(rng, 2, 64), lo=max(64, hi // 4), hi=hi, attn_out=rng.random() < 0.25)
    if kind == "recompute":
        hi = _log(rng, 1024, 16384)
        return dict(kind=kind, model=model, batch=_log(rng, 1, 64), lo=max(64, hi // 4), hi=hi, ratio=round(rng.uniform(0.01, 0.05), 3))
    if kind == "colsum":
        return dict(kind=kind, model=model, n=_log(rng, 512, 24000))
    if kind == "match":
        n = _log(rng, 1024, 131072)
        return dict(kind=kind, n=n, window=16 if n < 65536 else 32)
    return dict(kind="impact", model=model, n=_log(rng, 256, 7500))


# ---- inputs -------------------------------------------------------------------------------------------------------


def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(1_000_003 * seed + salt)


def _model(case):
    w = MODELS[case.get("model", "tiny")]
    if case["kind"] == "tiny":  # its spans take their listed share of whatever length is drawn
        w = synth.scaled(w, case["n"], span_lo=max(1, case["n"] // 16), span_hi=max(2, case["n"] // 4))
    elif case["kind"] in ("check", "recompute"):  # fully reused contexts
        w = synth.scaled(w, 0, coverage=1.0)
    else:
        w = synth.scaled(w, case["n"])
    return w


def _k(case):
    w = _model(case)
    return max(1, math.ceil(case["ratio"] * (w.coverage or 0.6) * case["n"]))


def _l1(a, b):
    """[heads, rows] L1 norms of a - b."""
    return (a.float() - b.float()).abs().sum(-1).t().contiguous()


def _picked(v_fresh, v_cache, reused, k):
    """Positions of the k reused tokens that deviate most, ascending."""
    s = _l1(v_fresh, v_cache).sum(0)
    s = torch.where(reused.bool(), s, torch.full_like(s, -1.0))
    return torch.topk(s, k).indices.sort().values.to(torch.int32)


def _layer(case, seed, layer=0, with_q=False):
    return synth.make_layer(_model(case), layer=layer, device=DEV, salt=seed, with_q=with_q)


def _workspace(call, shape, batch, rows, sel=0):
    return torch.empty(max(256, kvs.kvs_workspace_size(call, shape, batch, rows, sel)), dtype=torch.uint8, device=DEV)


def _inputs_attn(case, seed):
    a = _layer(case, seed, with_q=True)
    sel = _picked(a["v_fresh"], a["v_cache"], a["reused"], _k(case))
    at = sel.long()
    for c, f in (("k_cache", "k_fresh"), ("v_cache", "v_fresh")):
        a[c][at] = a[f][at]
    return dict(q=a["q"][at].contiguous(), sel=sel, k=a["k_cache"], v=a["v_cache"])


def _lengths(case):
    """The batch's context lengths: spread from lo to hi, in no order, the same for every seed."""
    r = random.Random(case["batch"] * 1_000_003 + case["lo"])
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]


def _inputs_batch(case, seed):
    """Packed caches of fully reused contexts, each with the decoding token's row appended."""
    w, gen = _model(case), _gen(seed, 17)
    length = _lengths(case)
    off = [sum(length[:b]) + b for b in range(case["batch"])]
    rows, new = sum(length) + case["batch"], torch.tensor([o + n for o, n in zip(off, length)], device=DEV)
    randn = lambda *shape: torch.randn(shape, generator=gen, device=DEV)  # noqa: E731
    sigma = torch.exp(w.sigma_mu + w.sigma_s * randn(rows))
    sigma[new] = 0.0
    fresh, cache = {}, {}
    for c in "kv":
        x = randn(rows, w.n_kv_heads, w.head_dim).to(w.torch_dtype)
        fresh[c] = x
        cache[c] = (x.float() + sigma[:, None, None] * randn(*x.shape)).to(w.torch_dtype)
    reused = torch.ones(rows, dtype=torch.uint8, device=DEV)
    reused[new] = 0
    q = (randn(case["batch"], w.n_q_heads, w.head_dim) / math.sqrt(w.head_dim)).to(w.torch_dtype)
    return dict(off=off, len=[n + 1 for n in length], q=q, k=cache["k"], v=cache["v"], dev_v=_l1(fresh["v"], cache["v"]), reused=reused,
                k_fresh=fresh["k"], v_fresh=fresh["v"])


def _inputs_project(case, seed, hidden, n_sel, layer=0):
    """Hidden states of the whole context, the fused weight, the rotary table."""
    w = _model(case)
    gen = _gen(seed, 11 + layer)
    x = torch.randn((w.n_ctx, hidden), generator=gen, device=DEV).to(torch.bfloat16)
    feats = (w.n_q_heads + 2 * w.n_kv_heads) * w.head_dim
    weight = (torch.randn((feats, hidden), generator=gen, device=DEV) / math.sqrt(hidden)).to(torch.bfloat16)
    rope = None
    if case.get("rope", True):
        rope = torch.from_numpy(synth.make_rope_table(w.n_ctx, w.head_dim)).to(DEV)
    return x, weight, rope


def _rows(case, seed):
    return torch.randperm(case["n"], generator=_gen(seed, 5), device=DEV)[: case["n_sel"]].sort().values.to(torch.int32)


def _outputs_project(w, n_sel):
    out = lambda h: torch.zeros((n_sel, h, w.head_dim), dtype=torch.bfloat16, device=DEV)  # noqa: E731
    return out(w.n_q_heads), out(w.n_kv_heads), out(w.n_kv_heads)


def _alpha(case, w, seed):
    """A column-mass profile like that of causal attention: what an earlier colsum call left."""
    if not case.get("alpha"):
        return None
    tail = torch.flip(torch.cumsum(torch.flip(1.0 / torch.arange(1, w.n_ctx + 1, device=DEV, dtype=torch.float64), [0]), 0), [0])
    return (w.group * tail.float() * (1.0 + torch.rand((w.n_kv_heads, w.n_ctx), generator=_gen(seed, 7), device=DEV))).contiguous()


def _attention64(q, sel, k, v, scale):
    """Exact causal attention of the rows `q` at positions `sel` over one context, (out, log-sum-exp)."""
    n_sel, hq, d = q.shape
    hk, grp = k.shape[1], q.shape[1] // k.shape[1]
    out = torch.empty((n_sel, hq, d), dtype=torch.float64, device=DEV)
    lse = torch.empty((n_sel, hq), dtype=torch.float64, device=DEV)
    step = max(1, 2048 // grp)
    for g in range(hk):
        for a in range(0, n_sel, step):
            e = min(n_sel, a + step)
            top = int(sel[e - 1]) + 1
            kg, vg = k[:top, g].double(), v[:top, g].double()
            s = (q[a:e, g * grp:(g + 1) * grp].double().reshape(-1, d) @ kg.t()).mul_(scale).view(e - a, grp, top)
            s.masked_fill_(torch.arange(top, device=DEV)[None, None] > sel[a:e, None, None].long(), -math.inf)
            z = torch.logsumexp(s, -1, keepdim=True)
            out[a:e, g * grp:(g + 1) * grp] = (s.sub_(z).exp_().view(-1, top) @ vg).view(e - a, grp, d)
            lse[a:e, g * grp:(g + 1) * grp] = z[..., 0]
    return out, lse


def _project64(x, weight, rope, rows, pos, w):
    y = (x[rows.long()].double() @ weight.double().t()).view(len(rows), -1, w.head_dim)
    if rope is not None:
        turned, half = w.n_q_heads + w.n_kv_heads, w.head_dim // 2
        c, s = rope[pos.long(), None, :, 0].double(), rope[pos.long(), None, :, 1].double()
        a, b = y[:, :turned, :half].clone(), y[:, :turned, half:].clone()
        y[:, :turned, :half] = a * c - b * s
        y[:, :turned, half:] = b * c + a * s
    return torch.split(y, [w.n_q_heads, w.n_kv_heads, w.n_kv_heads], 1)


def _top(score, k):
    return torch.sort(score.double(), descending=True, stable=True).indices[:k].sort().values.to(torch.int32)


def _colsum64(q, k, scale):
    n, hq, d = q.shape
    hk, grp = k.shape[1], hq // k.shape[1]
    alpha = torch.zeros((hk, n), dtype=torch.float64, device=DEV)
    for h in range(hq):
        kg = k[:, h // grp].double()
        for a in range(0, n, 4096):
            s = (q[a:a + 4096, h].double() @ kg.t()).mul_(scale)
            s.masked_fill_(torch.arange(n, device=DEV)[None] > torch.arange(a, a + len(s), device=DEV)[:, None], -math.inf)
            alpha[h // grp] += torch.softmax(s, -1).sum(0)
    return alpha


# ---- the cases ----------------------------------------------------------------------------------------------------


class Tiny:
    """Column mass, scores and selection on one layer; write-back and attention of the picked tokens on the next."""

    @staticmethod
    def prepare(case, seed):
        w, a, b = _model(case), _layer(case, seed, 0, True), _layer(case, seed, 1, True)
        n, k = case["n"], _k(case)
        shape = kvs.shape_of(w)
        zeros = lambda *s: torch.zeros(s, dtype=torch.float32, device=DEV)  # noqa: E731
        return dict(shape=shape, n=n, k=k, a=a, b=b, q=b["q"][:k].contiguous(), k_new=b["k_fresh"][:k].contiguous(), v_new=b["v_fresh"][:k].contiguous(),
                    k0=b["k_cache"].clone(), v0=b["v_cache"].clone(), alpha=zeros(w.n_kv_heads, n), dev_v=zeros(w.n_kv_heads, n), score=zeros(n),
                    idx=torch.zeros(k, dtype=torch.int32, device=DEV), out=zeros(k, w.n_q_heads, w.head_dim), lse=zeros(k, w.n_q_heads),
                    ws_alpha=_workspace("attn_colsum", shape, 1, n), ws=_workspace("partial_attention", shape, 1, n, k))

    @staticmethod
    def run(s):
        a, b, n, k = s["a"], s["b"], s["n"], s["k"]
        kvs.kvs_attn_colsum(s["shape"], n, a["q"], a["k_fresh"], 1.0, s["alpha"], s["ws_alpha"])
        kvs.kvs_deviation(s["shape"], n, None, a["v_fresh"], None, a["v_cache"], a["reused"], s["alpha"], kvs.SCORE_V, None, s["dev_v"], s["score"])
        kvs.kvs_select_topk(s["score"], [0, n], [k], s["idx"])
        kvs.kvs_scatter_kv(s["shape"], n, s["k_new"], s["v_new"], s["idx"], k, b["k_cache"], b["v_cache"])
        kvs.kvs_partial_attention(s["shape"], [0], [n], [0, k], s["q"], s["idx"], b["k_cache"], b["v_cache"], 1.0, s["out"], s["lse"], s["ws"])
        return dict(alpha=s["alpha"], dev_v=s["dev_v"], score=s["score"], idx=s["idx"], k_cache=b["k_cache"], v_cache=b["v_cache"], out=s["out"], lse=s["lse"])

    @staticmethod
    def work(case):
        w, n, k = _model(case), case["n"], _k(case)
        row, hq, hk, d = w.n_kv_heads * w.head_dim * 4, w.n_q_heads, w.n_kv_heads, w.head_dim
        return {"bytes": 3 * n * hq * d * 4 + 3 * n * row + 8 * k * row + 2 * k * hq * d * 4 + 8 * n * hk + 5 * n,
                "flops": 2 * d * hq * n * n // 2 + 4 * d * hq * k * n // 2}

    @staticmethod
    def tolerance(case):
        return {"rel": 2e-6, "max": 1e-4}  # fp32 sums of up to 2048 terms

    @staticmethod
    def exact(case, seed):
        s = Tiny.prepare(case, seed)
        a, b = s["a"], s["b"]
        alpha = _colsum64(a["q"], a["k_fresh"], 1.0)
        dev = (a["v_fresh"].double() - a["v_cache"].double()).abs().sum(-1).t()
        score = torch.where(a["reused"].bool(), (alpha * dev).sum(0), torch.full((s["n"],), -math.inf, dtype=torch.float64, device=DEV))
        idx = _top(score, s["k"])
        k, v = s["k0"].clone(), s["v0"].clone()
        k[idx.long()], v[idx.long()] = s["k_new"], s["v_new"]
        out, lse = _attention64(s["q"], idx, k, v, 1.0)
        return dict(alpha=alpha, dev_v=dev, score=score, idx=idx, k_cache=k.double(), v_cache=v.double(), out=out, lse=lse)


class Chain:
    """The check layer's selection, and the picked tokens' recomputation in a later layer with its index list."""

    @staticmethod
    def prepare(case, seed):
        w, a, b = _model(case), _layer(case, seed, 0), _layer(case, seed, 1)
        n, k = case["n"], _k(case)
        shape = kvs.shape_of(w)
        x, weight, rope = _inputs_project(case, seed, case["hidden"], k)
        q, kn, vn = _outputs_project(w, k)
        return dict(shape=shape, w=w, n=n, k=k, scale=1.0 / math.sqrt(w.head_dim), v_fresh=a["v_fresh"], v_cache0=a["v_cache"], reused=a["reused"],
                    k_cache=b["k_cache"], v_cache=b["v_cache"], x=x, weight=weight, rope=rope, q=q, k_new=kn, v_new=vn,
                    dev_v=torch.zeros((w.n_kv_heads, n), device=DEV), score=torch.zeros(n, device=DEV),
                    idx=torch.zeros(k, dtype=torch.int32, device=DEV), out=torch.zeros_like(q),
                    ws_top=_workspace("select_topk", shape, 1, n), ws=_workspace("partial_attention", shape, 1, n, k))

    @staticmethod
    def run(s):
        n, k = s["n"], s["k"]
        kvs.kvs_deviation_topk(s["shape"], n, None, s["v_fresh"], None, s["v_cache0"], s["reused"], None, kvs.SCORE_V, None, s["dev_v"], s["score"],
                               k, s["idx"], s["ws_top"])
        kvs.kvs_project_qkv(s["shape"], s["x"], s["idx"], s["idx"], k, s["weight"], s["rope"], s["q"], s["k_new"], s["v_new"])
        kvs.kvs_scatter_kv(s["shape"], n, s["k_new"], s["v_new"], s["idx"], k, s["k_cache"], s["v_cache"])
        kvs.kvs_partial_attention(s["shape"], [0], [n], [0, k], s["q"], s["idx"], s["k_cache"], s["v_cache"], s["scale"], s["out"], None, s["ws"])
        return dict(dev_v=s["dev_v"], score=s["score"], idx=s["idx"], k_cache=s["k_cache"], v_cache=s["v_cache"], out=s["out"])

    @staticmethod
    def work(case):
        parts = [Score.work(case), Project.work(dict(case, n_sel=_k(case), rope=True)), Attn.work(case)]
        w = _model(case)
        return {"bytes": sum(p["bytes"] for p in parts) + 4 * _k(case) * w.n_kv_heads * 256, "flops": sum(p["flops"] for p in parts)}

    @staticmethod
    def tolerance(case):
        return {"rel": 1.5e-2, "max": 0.3}  # bf16 results of a product enter a bf16 attention

    @staticmethod
    def exact(case, seed):
        s = Chain.prepare(case, seed)
        dev, score = Score.exact_scores(s["v_fresh"], s["v_cache0"], s["reused"])
        idx = _top(score.float(), s["k"])
        q, kn, vn = _project64(s["x"], s["weight"], s["rope"], idx, idx, s["w"])
        k, v = s["k_cache"].double(), s["v_cache"].double()
        k[idx.long()], v[idx.long()] = kn, vn
        return dict(dev_v=dev, score=score, idx=idx, k_cache=k, v_cache=v, out=_attention64(q, idx, k, v, s["scale"])[0])


class Score:
    """kvs_deviation_topk on one layer."""

    @staticmethod
    def prepare(case, seed):
        w, a = _model(case), _layer(case, seed)
        n, k = case["n"], _k(case)
        shape = kvs.shape_of(w)
        s = dict(shape=shape, n=n, k=k, mode=kvs.SCORE_KV if case["mode"] == "kv" else kvs.SCORE_V, reused=a["reused"], v_fresh=a["v_fresh"],
                 v_cache=a["v_cache"], k_fresh=None, k_cache=None, dev_k=None, alpha=_alpha(case, w, seed),
                 dev_v=torch.zeros((w.n_kv_heads, n), device=DEV), score=torch.zeros(n, device=DEV),
                 idx=torch.zeros(k, dtype=torch.int32, device=DEV), ws=_workspace("select_topk", shape, 1, n))
        if case["mode"] == "kv":
            s.update(k_fresh=a["k_fresh"], k_cache=a["k_cache"], dev_k=torch.zeros((w.n_kv_heads, n), device=DEV))
        return s

    @staticmethod
    def run(s):
        kvs.kvs_deviation_topk(s["shape"], s["n"], s["k_fresh"], s["v_fresh"], s["k_cache"], s["v_cache"], s["reused"], s["alpha"], s["mode"],
                               s["dev_k"], s["dev_v"], s["score"], s["k"], s["idx"], s["ws"])
        return dict(dev_k=s["dev_k"], dev_v=s["dev_v"], score=s["score"], idx=s["idx"])

    @staticmethod
    def work(case):
        w, n = _model(case), case["n"]
        sides = 2 if case.get("mode") == "kv" else 1
        per = sides * (2 * w.n_kv_heads * w.head_dim * 2 + 4 * w.n_kv_heads) + 1 + 4 + (4 * w.n_kv_heads if case.get("alpha") else 0)
        return {"bytes": per * n + 4 * _k(case), "flops": 3 * sides * n * w.n_kv_heads * w.head_dim}

    @staticmethod
    def tolerance(case):
        return {"rel": 5e-7, "max": 5e-6, "differ": 1e-3}  # fp32 sums of 128 terms, by head; a swap of near ties in the list

    @staticmethod
    def exact_scores(v_fresh, v_cache, reused, alpha=None, key=None):
        dev = (v_fresh.double() - v_cache.double()).abs().sum(-1).t()
        s = ((dev if key is None else key + dev) * (1.0 if alpha is None else alpha.double())).sum(0)
        return dev, torch.where(reused.bool(), s, torch.full_like(s, -math.inf))

    @staticmethod
    def exact(case, seed):
        s = Score.prepare(case, seed)
        key = (s["k_fresh"].double() - s["k_cache"].double()).abs().sum(-1).t() if case["mode"] == "kv" else None
        dev, score = Score.exact_scores(s["v_fresh"], s["v_cache"], s["reused"], s["alpha"], key)
        return dict(dev_k=key, dev_v=dev, score=score, idx=_top(score.float(), s["k"]))


class Attn:
    """kvs_partial_attention of one request's picked tokens, their rows written back already."""

    @staticmethod
    def prepare(case, seed):
        s = _inputs_attn(case, seed)
        w = _model(case)
        s.update(shape=kvs.shape_of(w), n=case["n"], n_sel=len(s["sel"]), out=torch.zeros_like(s["q"]))
        s["ws"] = _workspace("partial_attention", s["shape"], 1, s["n"], s["n_sel"])
        return s

    @staticmethod
    def run(s):
        kvs.kvs_partial_attention(s["shape"], [0], [s["n"]], [0, s["n_sel"]], s["q"], s["sel"], s["k"], s["v"], 1.0, s["out"], None, s["ws"])
        return s["out"]

    @staticmethod
    def work(case):
        w, n, k = _model(case), case["n"], _k(case)
        # the picked tokens are spread over the context: half of it lies before one, on average
        return {"bytes": 4 * n * w.n_kv_heads * w.head_dim + 4 * k * w.n_q_heads * w.head_dim + 4 * k, "flops": 4 * w.head_dim * w.n_q_heads * k * n // 2}

    @staticmethod
    def tolerance(case):
        return {"rel": 1e-2, "max": 0.2}  # softmax weights and results in bf16

    @staticmethod
    def exact(case, seed):
        s = _inputs_attn(case, seed)
        return _attention64(s["q"], s["sel"], s["k"], s["v"], 1.0)[0]


class Project:
    """kvs_project_qkv: Q, K and V of the picked tokens in a later layer."""

    @staticmethod
    def prepare(case, seed):
        w = _model(case)
        x, weight, rope = _inputs_project(case, seed, case["hidden"], case["n_sel"])
        q, k, v = _outputs_project(w, case["n_sel"])
        return dict(shape=kvs.shape_of(w), x=x, weight=weight, rope=rope, rows=_rows(case, seed), n_sel=case["n_sel"], q=q, k=k, v=v)

    @staticmethod
    def run(s):
        kvs.kvs_project_qkv(s["shape"], s["x"], s["rows"], s["rows"], s["n_sel"], s["weight"], s["rope"], s["q"], s["k"], s["v"])
        return s["q"], s["k"], s["v"]

    @staticmethod
    def work(case):
        w, m = _model(case), case["n_sel"]
        feats = (w.n_q_heads + 2 * w.n_kv_heads) * w.head_dim
        return {"bytes": 2 * case["hidden"] * (feats + m) + 2 * m * feats + (w.head_dim * 4 * m if case["rope"] else 0) + 4 * m,
                "flops": 2 * m * feats * case["hidden"]}

    @staticmethod
    def tolerance(case):
        return {"rel": 7e-3, "max": 2e-2}  # results in bf16

    @staticmethod
    def exact(case, seed):
        w, rows = _model(case), _rows(case, seed)
        x, weight, rope = _inputs_project(case, seed, case["hidden"], case["n_sel"])
        return tuple(_project64(x, weight, rope, rows, rows, w))


class Check:
    """kvs_decode_check: one decode step's re-check of a batch, 2 % of each context picked."""

    @staticmethod
    def prepare(case, seed):
        w, b = _model(case), _inputs_batch(case, seed)
        rows = b["k"].shape[0]
        k = [max(1, math.ceil(0.02 * n)) for n in b["len"]]
        shape = kvs.shape_of(w)
        return dict(shape=shape, rows=rows, off=b["off"], len=b["len"], q=b["q"], k=b["k"], v=b["v"] if case["attn_out"] else None, dev_v=b["dev_v"],
                    reused=b["reused"], k_req=k, idx=torch.zeros(sum(k), dtype=torch.int32, device=DEV), score=torch.zeros(rows, device=DEV),
                    out=torch.zeros_like(b["q"]) if case["attn_out"] else None, ws=_workspace("decode_check", shape, case["batch"], rows))

    @staticmethod
    def run(s):
        kvs.kvs_decode_check(s["shape"], s["rows"], s["off"], s["len"], s["q"], s["k"], s["v"], s["dev_v"], s["reused"], 1.0, s["k_req"], s["idx"],
                             s["score"], s["out"], s["ws"])
        return dict(idx=s["idx"], score=s["score"], out=s["out"])

    @staticmethod
    def work(case):
        w, rows = _model(case), sum(_lengths(case)) + case["batch"]
        sides = 2 if case["attn_out"] else 1
        return {"bytes": rows * (sides * w.n_kv_heads * w.head_dim * 2 + 4 * w.n_kv_heads + 5) + rows * 4 // 50,
                "flops": 2 * sides * rows * w.n_q_heads * w.head_dim}

    @staticmethod
    def tolerance(case):
        # scores: fp32 softmax of fp32 logits; a swap of near ties moves one request's list by a place
        return {"rel": 1e-2 if case["attn_out"] else 1e-6, "max": 0.1 if case["attn_out"] else 1e-4, "differ": 0.01}

    @staticmethod
    def exact(case, seed):
        w, b = _model(case), _inputs_batch(case, seed)
        rows, grp = b["k"].shape[0], w.group
        score = torch.zeros(rows, dtype=torch.float64, device=DEV)
        out = torch.zeros(b["q"].shape, dtype=torch.float64, device=DEV)
        idx = []
        for r, (o, n) in enumerate(zip(b["off"], b["len"])):
            s = torch.zeros(n, dtype=torch.float64, device=DEV)
            for g in range(w.n_kv_heads):
                p = torch.softmax(b["q"][r, g * grp:(g + 1) * grp].double() @ b["k"][o:o + n, g].double().t(), -1)
                s += p.sum(0) * b["dev_v"][g, o:o + n].double()
                if case["attn_out"]:
                    out[r, g * grp:(g + 1) * grp] = p @ b["v"][o:o + n, g].double()
            score[o:o + n] = torch.where(b["reused"][o:o + n].bool(), s, torch.full_like(s, -math.inf))
            idx.append(_top(score[o:o + n].float(), max(1, math.ceil(0.02 * n))))
        return dict(idx=torch.cat(idx), score=score, out=out if case["attn_out"] else None)


class Recompute:
    """What a decode step does with the picked tokens of its batch: write-back and attention."""

    @staticmethod
    def inputs(case, seed):
        w, b = _model(case), _inputs_batch(case, seed)
        sel, rows, cu = [], [], [0]
        dev = b["dev_v"].sum(0)
        for o, n in zip(b["off"], b["len"]):
            k = max(1, math.ceil(case["ratio"] * n))
            p = torch.topk(dev[o:o + n - 1], min(k, n - 1)).indices.sort().values
            sel.append(p)
            rows.append(p + o)
            cu.append(cu[-1] + len(p))
        sel, at = torch.cat(sel), torch.cat(rows)
        q = (torch.randn((len(sel), w.n_q_heads, w.head_dim), generator=_gen(seed, 3), device=DEV) / math.sqrt(w.head_dim)).to(w.torch_dtype)
        return dict(q=q, sel=sel.to(torch.int32), at=at.to(torch.int32), cu=cu, k_new=b["k_fresh"][at].contiguous(), v_new=b["v_fresh"][at].contiguous(),
                    k=b["k"], v=b["v"], reused=b["reused"], dev_v=b["dev_v"], off=b["off"], len=b["len"])

    @staticmethod
    def prepare(case, seed):
        s = Recompute.inputs(case, seed)
        w = _model(case)
        s.update(shape=kvs.shape_of(w), rows=s["k"].shape[0], n_sel=len(s["sel"]), out=torch.zeros_like(s["q"]))
        s["ws"] = _workspace("partial_attention", s["shape"], case["batch"], s["rows"], s["n_sel"])
        return s

    @staticmethod
    def run(s):
        kvs.kvs_scatter_kv(s["shape"], s["rows"], s["k_new"], s["v_new"], s["at"], s["n_sel"], s["k"], s["v"], s["reused"], s["dev_v"])
        kvs.kvs_partial_attention(s["shape"], s["off"], s["len"], s["cu"], s["q"], s["sel"], s["k"], s["v"], 1.0, s["out"], None, s["ws"])
        return dict(out=s["out"], k_cache=s["k"], v_cache=s["v"], reused=s["reused"], dev_v=s["dev_v"])

    @staticmethod
    def work(case):
        w, length = _model(case), _lengths(case)
        k = case["ratio"] * sum(length)
        row = w.n_kv_heads * w.head_dim * 2
        return {"bytes": int(2 * sum(length) * row + 4 * k * row + 4 * k * w.n_q_heads * w.head_dim + k * (9 + 4 * w.n_kv_heads)),
                "flops": int(4 * w.head_dim * w.n_q_heads * case["ratio"] * sum(n * n for n in length) / 2)}

    @staticmethod
    def tolerance(case):
        return {"rel": 1e-2, "max": 0.2}  # softmax weights and results in bf16

    @staticmethod
    def exact(case, seed):
        s = Recompute.inputs(case, seed)
        at = s["at"].long()
        s["k"][at], s["v"][at] = s["k_new"], s["v_new"]
        s["dev_v"][:, at] = 0
        outs = []
        for r, (o, n) in enumerate(zip(s["off"], s["len"])):
            a, e = s["cu"][r], s["cu"][r + 1]
            outs.append(_attention64(s["q"][a:e], s["sel"][a:e], s["k"][o:o + n], s["v"][o:o + n], 1.0)[0])
        return dict(out=torch.cat(outs), k_cache=None, v_cache=None, reused=None, dev_v=s["dev_v"].double())  # (the caches: rows copied)


class Colsum:
    """kvs_attn_colsum: the attention column mass of a whole prefill."""

    @staticmethod
    def prepare(case, seed):
        w, a = _model(case), _layer(case, seed, with_q=True)
        shape = kvs.shape_of(w)
        return dict(shape=shape, n=case["n"], q=a["q"], k=a["k_fresh"], alpha=torch.zeros((w.n_kv_heads, case["n"]), device=DEV),
                    ws=_workspace("attn_colsum", shape, 1, case["n"]))

    @staticmethod
    def run(s):
        kvs.kvs_attn_colsum(s["shape"], s["n"], s["q"], s["k"], 1.0, s["alpha"], s["ws"])
        return s["alpha"]

    @staticmethod
    def work(case):
        w, n = _model(case), case["n"]
        # every score is needed before a row's normaliser is known and again after it, or kept: one product counts
        return {"bytes": 2 * n * (w.n_q_heads + w.n_kv_heads) * w.head_dim + 4 * n * w.n_kv_heads, "flops": 2 * w.head_dim * w.n_q_heads * n * n // 2}

    @staticmethod
    def tolerance(case):
        return {"rel": 8e-6, "max": 1e-4}  # fp32 sums of up to 24000 softmax weights

    @staticmethod
    def exact(case, seed):
        a = _layer(case, seed, with_q=True)
        return _colsum64(a["q"], a["k_fresh"], 1.0)


class Match:
    """kvs_match_tokens: a new request's tokens against an earlier request's, with the ordered lists."""

    @staticmethod
    def prepare(case, seed):
        n = case["n"]
        st = synth.make_token_streams(synth.scaled(synth.LLAMA, n), seed=seed, window=case["window"], unique_candidate=False)
        ints = lambda: torch.zeros(n, dtype=torch.int32, device=DEV)  # noqa: E731
        return dict(target=torch.from_numpy(st["target"]).to(DEV), cand=torch.from_numpy(st["candidate"]).to(DEV), window=case["window"], match=ints(),
                    t=ints(), c=ints(), n=torch.zeros(1, dtype=torch.int64, device=DEV), ws=_workspace("match_tokens", None, 1, n, n))

    @staticmethod
    def run(s):
        kvs.kvs_match_tokens(s["target"], s["cand"], s["window"], HASH_BASE, HASH_MODULUS, s["match"], s["t"], s["c"], s["n"], s["ws"])
        return dict(match=s["match"], target=s["t"], candidate=s["c"], n=s["n"])

    @staticmethod
    def work(case):
        n = case["n"]
        return {"bytes": 4 * 5 * n, "flops": 2 * n * case["window"]}

    @staticmethod
    def tolerance(case):
        return "exact"

    @staticmethod
    def exact(case, seed):
        return None  # whole numbers


class Impact:
    """kvs_first_order_impact on a check layer."""

    @staticmethod
    def inputs(case, seed):
        a = _layer(case, seed, with_q=True)
        n, hq, d = a["q"].shape
        grp = hq // a["k_fresh"].shape[1]
        h = torch.empty_like(a["q"])
        lse = torch.empty((n, hq), dtype=torch.float32, device=DEV)
        for head in range(hq):  # the attention of every row over the fresh K and V, which the layer has computed
            k, v = a["k_fresh"][:, head // grp].float(), a["v_fresh"][:, head // grp].float()
            s = a["q"][:, head].float() @ k.t()
            s.masked_fill_(torch.triu(torch.ones((n, n), dtype=torch.bool, device=DEV), 1), -math.inf)
            z = torch.logsumexp(s, -1, keepdim=True)
            h[:, head] = (torch.exp(s - z) @ v).to(h.dtype)
            lse[:, head] = z[:, 0]
        a.update(h=h, lse=lse)
        return a

    @staticmethod
    def prepare(case, seed):
        a, w, n = Impact.inputs(case, seed), _model(case), case["n"]
        shape = kvs.shape_of(w)
        a.update(shape=shape, n=n, out=[torch.zeros(n, device=DEV) for _ in range(3)], ws=_workspace("first_order_impact", shape, 1, n))
        return a

    @staticmethod
    def run(s):
        kvs.kvs_first_order_impact(s["shape"], s["n"], s["q"], s["k_fresh"], s["v_fresh"], s["k_cache"], s["v_cache"], s["h"], s["lse"], s["reused"], 1.0,
                                   s["out"][0], s["out"][1], s["out"][2], s["ws"])
        return s["out"]

    @staticmethod
    def work(case):
        w, n = _model(case), case["n"]
        pairs = w.n_q_heads * n * (n + 1) // 2
        # two dot products a pair on the matrix cores; a difference, two norms and a product a channel besides
        return {"bytes": n * w.head_dim * 2 * (2 * w.n_q_heads + 4 * w.n_kv_heads) + 4 * n * w.n_q_heads + 13 * n, "flops": pairs * w.head_dim * 9}

    @staticmethod
    def tolerance(case):
        return {"rel": 1e-6, "max": 1e-4}  # fp32 sums

    @staticmethod
    def exact(case, seed):
        a = Impact.inputs(case, seed)
        n, hq, d = a["q"].shape
        grp = hq // a["k_fresh"].shape[1]
        imp = torch.zeros((3, n), dtype=torch.float64, device=DEV)
        step = 2048
        for head in range(hq):
            g = head // grp
            kf, vf = a["k_fresh"][:, g].double(), a["v_fresh"][:, g].double()
            dk, dv = a["k_cache"][:, g].double() - kf, a["v_cache"][:, g].double() - vf
            for r0 in range(0, n, step):  # rows of the attention matrix; the columns end with the last row's own
                r1 = min(n, r0 + step)
                q, h = a["q"][r0:r1, head].double(), a["h"][r0:r1, head].double()
                p = torch.exp(q @ kf[:r1].t() - a["lse"][r0:r1, head, None].double())
                p.masked_fill_(torch.arange(r1, device=DEV)[None] > torch.arange(r0, r1, device=DEV)[:, None], 0.0)
                t = q @ dk[:r1].t()
                key, both = torch.zeros_like(t), torch.zeros_like(t)
                for c in range(d):
                    x = vf[None, :r1, c] - h[:, c, None]
                    key += x.abs()
                    both += x.mul_(t).add_(dv[None, :r1, c]).abs_()
                imp[0, :r1] += p.sum(0) * dv[:r1].abs().sum(-1)
                imp[1, :r1] += (p * t.abs() * key).sum(0)
                imp[2, :r1] += (p * both).sum(0)
        return [torch.where(a["reused"].bool(), x, torch.full_like(x, -math.inf)) for x in imp]


KINDS = {"tiny": Tiny, "chain": Chain, "score": Score, "attn": Attn, "project": Project, "check": Check, "recompute": Recompute, "colsum": Colsum,
         "match": Match, "impact": Impact}


def prepare(case, seed):
    state = KINDS[case["kind"]].prepare(case, seed)
    state["kind"] = case["kind"]
    return state


def run(state):
    return KINDS[state["kind"]].run(state)


def work(case):
    return KINDS[case["kind"]].work(case)


def tolerance(case):
    return KINDS[case["kind"]].tolerance(case)


def exact(case, seed):
    return KINDS[case["kind"]].exact(case, seed)
