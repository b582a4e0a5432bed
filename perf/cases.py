"""The calls whose speed is measured: what a program that compresses KV caches has this library do.

A serving engine compresses layer by layer while it prefills (one layer, a handful of kv heads), or
a whole model's cache at once, or a batch of contexts of different lengths; it computes the
attention-based scores that the blend takes; it selects again on scores it has; it compacts into,
or inside, its page pool.  Sizes are those of the synthetic workloads (Llama-3.1-8B, Qwen-2.5-7B and
Qwen-2.5-32B head shapes, contexts of 4 K to 128 K tokens), odd ones among them.

Inputs.  Keys are the workloads' (outlier channels, low rank, rank deficiency).  In the fused calls
a share of every head's tokens equal to its retention is salient (rows four times as long, an exact
scaling in bf16), the rest is filler: retention is calibrated to what a context holds, and the kept
sets are then the same for any correct rounding of the scores, so that retained indices and packed
rows can be compared as they are.  Selection on its own runs on scores without such a gap.
"""
import math
import random

import torch

from paper_2507_08143_amd import compactor as C
from paper_2507_08143_amd import workloads as W

D = 128
GAIN = 4.0                      # length of a salient row over a filler row


def _case(name, op, **kw):
    c = {"name": name, "op": op, "layers": 1, "kv_heads": 8, "n": 0, "ratio": 0.3, "requests": 1,
         "shape_seed": 0, "n_lo": 0, "sketch": 48, "ridge": 0.0, "keys": "outlier", "layout": "head",
         "scope": "head", "blend": False, "group": 4, "page": 16}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest fused call: one head of a short context, all latency
        _case("compress_head_4k", "compress", kv_heads=1, n=4096, ratio=0.5),
        # one layer of a Llama-3.1-8B prefill, as an engine compresses it when the layer is done
        _case("compress_layer_8k", "compress", n=8192, keys="lowrank"),
        # the same at the long end of the context range
        _case("compress_layer_128k", "compress", n=131072, ratio=0.2),
        # the whole cache of a Llama-3.1-8B context in one call
        _case("compress_model_32k", "compress", layers=32, n=32768, keys="lowrank"),
        # contexts of different lengths with calibrated retention, cache kept token by token
        _case("compress_ragged_batch", "compress", layers=2, requests=12, n_lo=8192, n=65536,
              shape_seed=4, layout="token"),
        # exact leverage scores with a ridge on rank-deficient keys, some layers of Qwen-2.5-32B
        _case("compress_exact_50k", "compress", layers=4, n=50001, ratio=0.32, sketch=0, ridge=1e-4,
              keys="deficient"),
        # the full method's second half: blend with attention scores, budget shared by a layer's heads
        _case("compress_blend_scope_16k", "compress", layers=4, n=16383, blend=True, scope="layer"),
        # scores alone (a caller with a selection of its own), Qwen-2.5-7B heads, token-major cache
        _case("score_layers_40k", "score", layers=2, kv_heads=4, n=40007, sketch=32, layout="token"),
        # attention scores of one layer of a short context, and of some layers of a long one
        _case("attention_layer_4k", "attention", n=4095),
        _case("attention_layers_32k", "attention", layers=4, n=32768),
        # selection on existing scores, all heads of a Qwen-2.5-7B context
        _case("select_model_128k", "select", layers=28, kv_heads=4, n=131072, ratio=0.2),
        # a paged cache compacted where it lies, some layers of a context
        _case("paged_in_place_16k", "in_place", layers=4, n=16384),
    ]


ROWS_MOST = 32 * 8 * 32768      # head-rows of the largest listed call
ATT_ROWS_MOST = 4 * 8 * 32768


def draw(rng):
    op = rng.choice(["compress"] * 6 + ["score", "attention", "attention", "select", "select",
                                        "paged", "in_place", "compact"])
    kv = rng.choice([1, 2, 4, 8, 8])
    most = ATT_ROWS_MOST if op == "attention" else ROWS_MOST
    n = int(round(math.exp(rng.uniform(math.log(1024), math.log(131072)))))
    if rng.random() < 0.3:
        n = max(1024, n // 256 * 256)
    layers = int(round(math.exp(rng.uniform(0.0, math.log(max(1.0, min(32.0, most / (kv * n))))))))
    c = _case("", op, layers=max(1, layers), kv_heads=kv, n=n, ratio=round(rng.uniform(0.1, 0.6), 3),
              layout=rng.choice(["head", "head", "token"]))
    if op in ("compress", "score"):
        mode = rng.choice(["sketch", "sketch", "sketch", "exact"])
        if mode == "exact":
            c.update(sketch=0, ridge=1e-4, keys="deficient")
        else:
            c.update(sketch=rng.choice([16, 32, 48, 48, 64]), keys=rng.choice(["outlier", "lowrank"]))
            if c["keys"] == "lowrank":
                c["sketch"] = min(c["sketch"], 48)
    if op == "compress":
        c.update(blend=rng.random() < 0.3, scope=rng.choice(["head", "head", "layer"]))
        if rng.random() < 0.25:
            c.update(requests=rng.randint(2, 12), n_lo=max(1024, n // 8), shape_seed=rng.randint(1, 10**6))
            while c["layers"] > 1 and c["layers"] * kv * n * c["requests"] > ROWS_MOST:
                c["layers"] //= 2
            while c["requests"] > 2 and c["layers"] * kv * n * c["requests"] > ROWS_MOST:
                c["requests"] -= 1
    if op in ("select", "paged", "compact"):
        c["scope"] = rng.choice(["head", "head", "layer"])
    if op in ("paged", "in_place"):
        c["page"] = rng.choice([16, 32, 64, 256])
    if op == "attention":
        c["group"] = rng.choice([1, 2, 4, 4, 7])
        while c["layers"] > 1 and c["layers"] * kv * n * c["group"] > 4 * ATT_ROWS_MOST:
            c["layers"] //= 2
    del c["name"]
    return c


def _shapes(case):
    """(tokens, retention) of every request of the call."""
    if case["requests"] == 1:
        return [(case["n"], case["ratio"])]
    r = random.Random(case["shape_seed"])
    return [(r.randint(case["n_lo"], case["n"]), round(r.uniform(0.2, 0.6), 3))
            for _ in range(case["requests"])]


def _laid_out(t, layout):
    """[L, H, n, d] as the cache holds it: head by head, or token by token."""
    if layout == "head":
        return t
    return t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)


def _salient(case, n, k, g, dev):
    """bool [L, H, n]: k tokens of every head, or H*k of every layer wherever they fall."""
    L, H = case["layers"], case["kv_heads"]
    m = torch.zeros(L, H, n, dtype=torch.bool, device=dev)
    for l in range(L):
        if case["scope"] == "layer":
            m[l].view(-1)[torch.rand(H * n, generator=g, device=dev).topk(H * k).indices] = True
        else:
            m[l].scatter_(1, torch.rand(H, n, generator=g, device=dev).topk(k, dim=1).indices, True)
    return m


def _keys(kind, L, H, n, g, dev):
    if kind == "lowrank":
        return W.lowrank_outlier_keys(L, H, n, D, g, dev)
    if kind == "deficient":
        return W.rank_deficient_duplicate_keys(L, H, n, D, g, dev, dup_frac=0.0)
    return W.gaussian_outlier_keys(L, H, n, D, g, dev)


def _inputs(case, seed):
    """Keys, values and attention scores of a compress or score call, one triple per request."""
    dev = torch.device("cuda", torch.cuda.current_device())
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 1000003 + 17)
    L, H = case["layers"], case["kv_heads"]
    got = []
    for n, ratio in _shapes(case):
        k = _keys(case["keys"], L, H, n, g, dev)
        m = _salient(case, n, C.compactor_keep_count(n, ratio), g, dev)
        k *= torch.where(m, GAIN, 1.0).to(torch.bfloat16).unsqueeze(-1)
        v = W._values(L, H, n, D, g, dev) if case["op"] == "compress" else k
        a = None
        if case["blend"]:       # column sums of a softmax average to 1; salient tokens draw more
            a = (0.5 + torch.rand(L, H, n, generator=g, device=dev)) * torch.where(m, 6.0, 1.0)
        got.append((_laid_out(k, case["layout"]), _laid_out(v, case["layout"]), a))
    return got


def _phi(case, dev):
    return W.make_phi(ks=case["sketch"], device=dev) if case["sketch"] > 0 else None


def _params(case, dev):
    return C.Params(case["layers"], case["kv_heads"], sketch_dim=case["sketch"], phi=_phi(case, dev),
                    ridge_rel=case["ridge"], lambda_blend=W.LAMBDA_BLEND,
                    select_scope=C.SCOPE_LAYER if case["scope"] == "layer" else C.SCOPE_HEAD)


def _workspace(p, reqs, dev):
    """A program allocates its scratch once and passes it to every call."""
    return torch.empty(max(256, C.compactor_workspace_size(p, reqs)), dtype=torch.uint8, device=dev)


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    op, L, H = case["op"], case["layers"], case["kv_heads"]
    if op in ("compress", "score"):
        p = _params(case, dev)
        reqs = [C.Request(k_score=k, v_cache=v, ratio=r, attn=a)
                for (k, v, a), (_, r) in zip(_inputs(case, seed), _shapes(case))]
        return {"op": op, "p": p, "reqs": reqs, "ws": _workspace(p, reqs, dev)}
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 1000003 + 23)
    n = case["n"]
    if op == "attention":
        k = W.gaussian_outlier_keys(L, H, n, D, g, dev)
        q = W.synthetic_queries(L, H * case["group"], n, device=dev, seed=seed)
        p = C.AttnParams(L, H, H * case["group"])
        reqs = [C.AttnRequest(q=_laid_out(q, case["layout"]), k=_laid_out(k, case["layout"]))]
        ws = torch.empty(max(256, C.compactor_attention_workspace_size(p, reqs)), dtype=torch.uint8,
                         device=dev)
        return {"op": op, "p": p, "reqs": reqs, "ws": ws}
    # selection and compaction: leverage-like scores (sums of k_s squares over n)
    p = _params(case, dev)
    scores = torch.randn(L * H * n, generator=g, device=dev)
    scores = (1.0 + 0.2 * scores).clamp_(min=0.05).mul_(W.SKETCH_DIM / n)
    if op in ("select", "in_place"):          # no dense cache is read: a view that only says the sizes
        k = v = torch.zeros(1, 1, 1, D, dtype=torch.bfloat16, device=dev).expand(L, H, n, D)
    else:
        k = _laid_out(W._values(L, H, n, D, g, dev), case["layout"])
        v = _laid_out(W._values(L, H, n, D, g, dev), case["layout"])
    reqs = [C.Request(k_score=k, v_cache=v, ratio=case["ratio"])]
    s = {"op": op, "p": p, "reqs": reqs, "ws": _workspace(p, reqs, dev), "scores": scores}
    if op == "select":
        return s
    s["kept"], s["cnt"] = C.compactor_select(p, reqs, scores, workspace=s["ws"])
    if op == "compact":
        return s
    # a page pool per layer, [page][slot][head][channel], pages dealt at random
    kk = C.compactor_keep_count(n, case["ratio"])
    rows = n if op == "in_place" else (min(n, H * kk) if case["scope"] == "layer" else kk)
    pages = -(-rows // case["page"])
    pool = pages + pages // 8 + 1
    s["table"] = torch.randperm(pool, generator=g, device=dev)[:pages].to(torch.int32)
    for name in ("k_pages", "v_pages"):
        t = torch.zeros(L, pool, case["page"], H, D, dtype=torch.bfloat16, device=dev)
        if op == "in_place":
            for l in range(L):
                t[l] = torch.randn(t[l].shape, generator=g, device=dev).to(torch.bfloat16)
        s[name] = t.permute(1, 0, 2, 3, 4)
    return s


def _bits(t):
    """Packed rows and pages are bit copies: compared as whole values."""
    return t.view(torch.int16)


def run(s):
    op, p, reqs = s["op"], s["p"], s["reqs"]
    if op == "compress":
        o = C.compactor_compress(p, reqs, want_scores=True, workspace=s["ws"])
        return {"scores": o["scores"], "kept_idx": o["kept_idx"], "kept_cnt": o["kept_cnt"],
                "status": o["status"], "k_packed": _bits(o["k_packed"]), "v_packed": _bits(o["v_packed"])}
    if op == "score":
        scores, status = C.compactor_score(p, reqs, workspace=s["ws"])
        return {"scores": scores, "status": status}
    if op == "attention":
        return C.compactor_attention_scores(p, reqs, workspace=s["ws"])
    if op == "select":
        kept, cnt = C.compactor_select(p, reqs, s["scores"], workspace=s["ws"])
        return {"kept_idx": kept, "kept_cnt": cnt}
    if op == "compact":
        k, v = C.compactor_compact(p, reqs, s["kept"], s["cnt"])
        return {"k_packed": _bits(k), "v_packed": _bits(v)}
    C.compactor_compact_paged(p, reqs, s["kept"], s["cnt"], s["k_pages"], s["v_pages"], [s["table"]],
                              in_place=op == "in_place")
    return {"k_pages": _bits(s["k_pages"]), "v_pages": _bits(s["v_pages"])}


def work(case):
    LH = case["layers"] * case["kv_heads"]
    rows = LH * sum(n for n, _ in _shapes(case))
    kept = LH * sum(C.compactor_keep_count(n, r) for n, r in _shapes(case))
    op, ks = case["op"], case["sketch"]
    # sketching a row, its share of the small Gram matrix and its quadratic form
    per_row = 2 * D * ks + 3 * ks * ks if ks > 0 else 2 * D * D
    if op == "score":
        return {"bytes": rows * (2 * D + 4), "flops": rows * per_row}
    if op == "compress":     # K read once, V where retained; scores, indices and packed rows written
        return {"bytes": rows * (2 * D + 4 + (4 if case["blend"] else 0)) + kept * (4 + 6 * D),
                "flops": rows * per_row}
    if op == "attention":
        last = case["n"] % 256
        pairs = case["n"] // 256 * 256 * 256 + last * last
        G = case["group"]
        return {"bytes": rows * (2 * D * (1 + G) + 4), "flops": LH * G * pairs * 2 * D}
    if op == "select":
        return {"bytes": rows * 4 + kept * 4, "flops": 0}
    return {"bytes": kept * (4 + 8 * D), "flops": 0}


def tolerance(case):
    """About four times the difference, over the ranges, from 64 bits and from the same sums in
    another partition."""
    op = case["op"]
    if op == "attention":       # fp32 softmax and sums
        return {"rel": 4e-7, "max": 2e-6}
    if op not in ("compress", "score"):
        return "exact"
    # fp32 accumulation of the Gram matrix carried through its inverse (keys of low rank are the
    # worse conditioned ones), W^T with 16 mantissa bits; a blend adds z(a), which is exact
    rel = {"outlier": 5e-6, "lowrank": 3.5e-5, "deficient": 4.5e-5}[case["keys"]]
    rel = rel / 3 if case["blend"] else rel
    return {"rel": rel, "max": 8 * rel}


def exact(case, seed):
    op, L, H = case["op"], case["layers"], case["kv_heads"]
    dev = torch.device("cuda", torch.cuda.current_device())
    if op == "attention":
        st = prepare(case, seed)
        q, k = st["reqs"][0].q, st["reqs"][0].k
        n, G = case["n"], case["group"]
        out = torch.zeros(L, H, n, dtype=torch.float64, device=dev)
        for l in range(L):
            for h in range(H):
                for j in range(G):
                    for c0, blocks, C0 in ((0, n // 256, 256), (n // 256 * 256, 1, n % 256)):
                        if blocks == 0 or C0 == 0:
                            continue
                        e = c0 + blocks * C0
                        qb = q[l, h * G + j, c0:e].double().reshape(blocks, C0, D)
                        kb = k[l, h, c0:e].double().reshape(blocks, C0, D)
                        x = torch.bmm(qb, kb.transpose(1, 2).contiguous()) / math.sqrt(D)
                        out[l, h, c0:e] += torch.softmax(x, dim=2).sum(1).reshape(-1) / G
        pool = st["p"].pool
        pad = torch.nn.functional.pad(out, (pool // 2, pool // 2))
        return sum(pad[..., i:i + n] for i in range(pool)).reshape(-1) / pool
    if op not in ("compress", "score"):
        return None
    phi = _phi(case, dev)
    phi = phi.double() if phi is not None else None
    parts = []
    for k, _, a in _inputs(case, seed):
        for l in range(L):
            for h in range(H):
                x = k[l, h].double()
                x = x @ phi if phi is not None else x
                S = x.t() @ x
                S = S + case["ridge"] * S.trace() / S.shape[0] * torch.eye(S.shape[0], dtype=S.dtype, device=dev)
                o = torch.linalg.solve_triangular(torch.linalg.cholesky(S), x.t().contiguous(), upper=False)
                o = o.square().sum(0)
                if a is not None:
                    z = lambda t: (t - t.mean()) / t.std(unbiased=False)  # noqa: E731
                    o = z(a[l, h].double()) + W.LAMBDA_BLEND * z(o)
                parts.append(o)
    out = {"scores": torch.cat(parts), "status": None}
    if op == "compress":
        out.update(kept_idx=None, kept_cnt=None, k_packed=None, v_packed=None)
    return out
