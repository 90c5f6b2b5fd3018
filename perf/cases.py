"""Performance cases of the layerwise prefix-KV path.

Each case is one piece of work a serving program hands the library through
its Python entry points: a layer's suffix attention, a layer's ingest, a
request's chunk objects in and out, the rest of a layer, or a whole pipeline
run.  `listed()` names the representative ones, `draw()` gives more of the
same ranges.  Inputs are N(0, 1) bfloat16 from the seed, block tables random
permutations of the pool's pages.
"""
import math
import random

import torch

import paper_2605_22850_amd as oc

PAGE = 16
DEV = "cuda"


def listed():
    return [
        # The smallest layer: the tiny workload (256 cached tokens, 32 new
        # ones), all launch latency.
        {"name": "attn_tiny", "kind": "attention", "nq": 4, "nkv": 2, "d": 64, "prefix": 256, "suffix": 32,
         "static_ws": False},
        # A prompt found whole in the cache: only its last token is computed,
        # so the layer streams the prefix through one query row per head (the
        # prefix ends inside a page).
        {"name": "attn_full_hit", "kind": "attention", "nq": 32, "nkv": 8, "d": 128, "prefix": 32763, "suffix": 1,
         "static_ws": False},
        # An ordinary hit on the 8B shape: 4K cached, a short question behind
        # it (the 8b-4k workload's layer).
        {"name": "attn_8b_4k", "kind": "attention", "nq": 32, "nkv": 8, "d": 128, "prefix": 4096, "suffix": 128,
         "static_ws": False},
        # A 4K context with a 12.5 % hit: a short cached prefix and a long
        # causal suffix (the first end-to-end cell).
        {"name": "attn_8b_4k_miss", "kind": "attention", "nq": 32, "nkv": 8, "d": 128, "prefix": 512, "suffix": 3584,
         "static_ws": False},
        # The long-context layer (the 8b-64k workload), bound by the
        # matrix cores.
        {"name": "attn_8b_64k", "kind": "attention", "nq": 32, "nkv": 8, "d": 128, "prefix": 65536, "suffix": 512,
         "static_ws": False},
        # The 70B shape's layer: eight query heads to a KV head, called
        # without a workspace as code under capture does.
        {"name": "attn_70b_32k", "kind": "attention", "nq": 64, "nkv": 8, "d": 128, "prefix": 32768, "suffix": 512,
         "static_ws": True},
        # The smallest layer payload (the tiny workload's), launch latency.
        {"name": "ingest_tiny", "kind": "ingest", "nkv": 2, "d": 64, "page": 16, "chunk": 16, "prefix": 256},
        # The long-context layer payload: 256 MiB unpacked and scattered.
        {"name": "ingest_8b_64k", "kind": "ingest", "nkv": 8, "d": 128, "page": 16, "chunk": 16, "prefix": 65536},
        # A request's chunk objects under chunkwise delivery and write-back:
        # whole objects of 64 tokens scattered into every layer, the suffix
        # appended layer by layer, the new whole chunks gathered back.
        {"name": "chunk_objects_4k", "kind": "chunk_objects", "layers": 32, "nkv": 8, "d": 128, "chunk": 64,
         "prefix": 4096, "suffix": 512},
        # What an 8B layer runs on the miss tokens besides the attention.
        {"name": "rest_of_layer_128", "kind": "rest_of_layer", "nq": 32, "nkv": 8, "d": 128, "ffn": 14336,
         "tokens": 128},
        # Eight requests with 5K to 28K cached tokens and 256 new ones share
        # a pool; payloads already in device memory, ingest overlapped with
        # attention, suffix appended (the batch workload, eight layers of it).
        {"name": "staged_batch8", "kind": "pipeline", "mode": "staged", "layers": 8, "nq": 32, "nkv": 8, "d": 128,
         "chunk": 16, "prefixes": "22288 11664 12704 11440 4992 6512 28560 8144", "suffix": 256, "append": True},
        # One 4K request from the host producer at the host link's full
        # rate, all 32 layers of the 8B shape.
        {"name": "producer_8b_4k", "kind": "pipeline", "mode": "producer", "layers": 32, "nq": 32, "nkv": 8, "d": 128,
         "chunk": 16, "prefixes": "4096", "suffix": 128, "append": False},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attention"] * 6 + ["ingest"] * 2 + ["chunk_objects", "rest_of_layer"] + ["pipeline"] * 2)
    if kind == "attention":
        while True:
            nq, nkv, d = rng.choice([(4, 2, 64), (8, 8, 64), (32, 8, 128), (32, 8, 128), (64, 8, 128), (4, 1, 128),
                                     (32, 4, 64)])
            case = {"kind": kind, "nq": nq, "nkv": nkv, "d": d, "prefix": _log_uniform(rng, 16, 65536),
                    "suffix": _log_uniform(rng, 1, 3584), "static_ws": rng.random() < 0.3}
            if work(case)["flops"] < 1e12:
                return case
    if kind == "ingest":
        nkv, d = rng.choice([(2, 64), (8, 128), (8, 128), (1, 128), (3, 96)])
        chunk = rng.choice([16, 16, 64, 256, 24])
        return {"kind": kind, "nkv": nkv, "d": d, "page": rng.choice([16, 16, 32, 24]), "chunk": chunk,
                "prefix": chunk * max(1, _log_uniform(rng, 64, 65536) // chunk)}
    if kind == "chunk_objects":
        chunk = rng.choice([16, 64, 256])
        return {"kind": kind, "layers": rng.randint(2, 32), "nkv": rng.choice([2, 8]), "d": rng.choice([64, 128]),
                "chunk": chunk, "prefix": chunk * max(1, _log_uniform(rng, 256, 4096) // chunk),
                "suffix": chunk * rng.randint(1, 3) + rng.randint(0, 15)}
    if kind == "rest_of_layer":
        nq, nkv, d, ffn = rng.choice([(32, 8, 128, 14336), (32, 8, 128, 14336), (8, 2, 64, 1792)])
        return {"kind": kind, "nq": nq, "nkv": nkv, "d": d, "ffn": ffn, "tokens": _log_uniform(rng, 1, 3584)}
    nq, nkv, d = rng.choice([(32, 8, 128), (32, 8, 128), (4, 2, 64)])
    n = rng.randint(1, 8)
    prefixes = [16 * (_log_uniform(rng, 256, 16384) // 16) for _ in range(n)]
    return {"kind": kind, "mode": "staged", "layers": rng.randint(2, 8), "nq": nq, "nkv": nkv, "d": d, "chunk": 16,
            "prefixes": " ".join(str(p) for p in prefixes), "suffix": _log_uniform(rng, 8, 256),
            "append": rng.random() < 0.5}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, *shape, scale=1.0):
    x = torch.randn(*shape, dtype=torch.bfloat16, device=DEV, generator=g)
    return x if scale == 1.0 else x.mul_(scale)


def _pages(n_tokens, page=PAGE):
    return -(-n_tokens // page)


def _tables(g, needs, pool_pages):
    """Disjoint random tables over one pool, one per request."""
    perm = torch.randperm(pool_pages, device=DEV, generator=g).to(torch.int32)
    out, at = [], 0
    for n in needs:
        out.append(perm[at:at + n].clone())
        at += n
    return out


def _attention(case, seed):
    g = _gen(seed)
    nq, nkv, d, tp, ts = (case[k] for k in ("nq", "nkv", "d", "prefix", "suffix"))
    need = _pages(tp)
    lay = oc.Layout(1, nq, nkv, d, PAGE, 16, 4 * need)
    pool = _normal(g, lay.pool_elems)
    table, = _tables(g, [need], lay.num_pages)
    q, k, v = _normal(g, ts, nq, d), _normal(g, ts, nkv, d), _normal(g, ts, nkv, d)
    return lay, pool, table, q, k, v


def _objects_shape(case, tokens):
    return tokens // case["chunk"], case["layers"], 2, case["chunk"], case["nkv"], case["d"]


def _chunk_objects(case, seed):
    g = _gen(seed)
    tp, ts, L = case["prefix"], case["suffix"], case["layers"]
    need = _pages(tp + ts)
    lay = oc.Layout(L, case["nkv"], case["nkv"], case["d"], PAGE, case["chunk"], need + need // 4)
    objects = _normal(g, *_objects_shape(case, tp))
    k, v = _normal(g, L, ts, case["nkv"], case["d"]), _normal(g, L, ts, case["nkv"], case["d"])
    table, = _tables(g, [need], lay.num_pages)
    return lay, objects, k, v, table


def _layer(case, seed):
    g = _gen(seed)
    H, F, n_qkv = case["nq"] * case["d"], case["ffn"], (case["nq"] + 2 * case["nkv"]) * case["d"]
    x = _normal(g, case["tokens"], H)
    w = [_normal(g, 1, K, N, scale=K ** -0.5) for K, N in ((H, H), (H, 2 * F), (F, H), (H, n_qkv))]
    return x, w


def _pipeline(case, seed):
    g = _gen(seed)
    L, nq, nkv, d, G, ts = (case[k] for k in ("layers", "nq", "nkv", "d", "chunk", "suffix"))
    tps = [int(x) for x in case["prefixes"].split()]
    needs = [_pages(t + ts) for t in tps]
    lay = oc.Layout(L, nq, nkv, d, PAGE, G, sum(needs) + sum(needs) // 4)
    tables = _tables(g, needs, lay.num_pages)
    reqs = []
    for t in tps:
        # payloads [layer][chunk][K|V][token][head][dim]
        kv = _normal(g, L, t // G, 2, G, nkv, d)
        reqs.append((kv, _normal(g, L, ts, nq, d), _normal(g, L, ts, nkv, d), _normal(g, L, ts, nkv, d)))
    return lay, tables, tps, reqs


class _Context:
    """A pipeline context, destroyed with the object."""

    def __init__(self, *a, **kw):
        self.ctx = oc.oc_context_create(*a, **kw)

    def __del__(self):
        oc.oc_context_destroy(self.ctx)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "attention":
        lay, pool, table, q, k, v = _attention(case, seed)
        ws = None
        if not case["static_ws"]:
            ws = torch.empty(oc.oc_attention_workspace_bytes(lay, case["prefix"], case["suffix"]), dtype=torch.uint8,
                             device=DEV)
        return {"case": case, "lay": lay, "pool": pool, "table": table, "q": q, "k": k, "v": v,
                "out": torch.empty_like(q), "ws": ws}
    if kind == "ingest":
        g = _gen(seed)
        tp, need = case["prefix"], _pages(case["prefix"], case["page"])
        lay = oc.Layout(1, case["nkv"], case["nkv"], case["d"], case["page"], case["chunk"], 4 * need)
        payload = _normal(g, tp // case["chunk"], 2, case["chunk"], case["nkv"], case["d"])
        table, = _tables(g, [need], lay.num_pages)
        return {"case": case, "lay": lay, "payload": payload, "table": table,
                "pool": torch.zeros(lay.pool_elems, dtype=torch.bfloat16, device=DEV)}
    if kind == "chunk_objects":
        lay, objects, k, v, table = _chunk_objects(case, seed)
        tokens = case["prefix"] + case["suffix"]
        first = case["prefix"] // case["chunk"]
        fresh = torch.empty(_objects_shape(case, tokens - case["prefix"]), dtype=torch.bfloat16, device=DEV)
        return {"case": case, "lay": lay, "objects": objects, "k": k, "v": v, "table": table, "first": first,
                "fresh": fresh, "pool": torch.zeros(lay.pool_elems, dtype=torch.bfloat16, device=DEV)}
    if kind == "rest_of_layer":
        x, w = _layer(case, seed)
        lay = oc.Layout(1, case["nq"], case["nkv"], case["d"], PAGE, 16, 1)
        T, H, F = case["tokens"], case["nq"] * case["d"], case["ffn"]
        bufs = [torch.empty(T, n, dtype=torch.bfloat16, device=DEV)
                for n in (H, 2 * F, F, H, (case["nq"] + 2 * case["nkv"]) * case["d"])]
        return {"case": case, "lay": lay, "x": x, "w": oc.LayerWeights(F, *w), "bufs": bufs}
    lay, tables, tps, reqs = _pipeline(case, seed)
    pool = torch.zeros(lay.pool_elems, dtype=torch.bfloat16, device=DEV)
    staged = case["mode"] == "staged"
    requests = []
    for t, table, (kv, q, k, v) in zip(tps, tables, reqs):
        if staged:
            src = {"device_payload": kv}
        else:
            # chunk objects as stored: every layer of a chunk together
            objects = kv.transpose(0, 1).contiguous().reshape(t // lay.chunk_tokens, -1)
            src = {"chunk_objects": objects.view(torch.int16).cpu().numpy()}
        requests.append(oc.Request(t, case["suffix"], table, q, k, v, torch.empty_like(q), **src))
    torch.cuda.synchronize()
    ctx = _Context(pool, lay, oc.OC_MODE_DEVICE_STAGED if staged else oc.OC_MODE_PRODUCER, max(tps), case["suffix"],
                   append_suffix=case["append"])
    return {"case": case, "lay": lay, "pool": pool, "requests": requests, "ctx": ctx}


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    case, lay = s["case"], s["lay"]
    kind = case["kind"]
    if kind == "attention":
        args = (s["q"], s["k"], s["v"], case["suffix"], s["pool"], lay, s["table"], case["prefix"], 0, s["out"])
        if s["ws"] is None:
            oc.oc_suffix_prefill_layer_noalloc(*args)
        else:
            oc.oc_suffix_prefill_layer(*args, s["ws"])
        return s["out"]
    if kind == "ingest":
        oc.oc_kv_layer_ingest(s["payload"], case["prefix"] // case["chunk"], s["table"], case["prefix"], s["pool"],
                              lay, 0)
        return s["pool"].view(torch.int16)
    if kind == "chunk_objects":
        tp, ts = case["prefix"], case["suffix"]
        oc.oc_kv_chunks_ingest(s["objects"], s["first"], 0, s["table"], tp, s["pool"], lay)
        for layer in range(case["layers"]):
            oc.oc_kv_suffix_append(s["k"][layer], s["v"][layer], ts, s["table"], tp, s["pool"], lay, layer)
        oc.oc_kv_chunks_gather(s["table"], tp + ts, s["pool"], lay, s["first"], (tp + ts) // case["chunk"] - s["first"],
                               s["fresh"])
        return {"pool": s["pool"].view(torch.int16), "objects": s["fresh"].view(torch.int16)}
    if kind == "rest_of_layer":
        oc.oc_rest_of_layer(s["x"], case["tokens"], lay, s["w"], 0, *s["bufs"])
        return s["bufs"]
    oc.oc_pipeline_run(s["ctx"].ctx, s["requests"], case["layers"])
    return {"out": [r.out for r in s["requests"]], "pool": s["pool"].view(torch.int16)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _attention_work(nq, nkv, d, tp, ts):
    return (2 * d * (2 * nq * ts + 2 * nkv * (tp + ts)), 4 * nq * d * (ts * tp + ts * (ts + 1) // 2))


def work(case):
    kind = case["kind"]
    if kind == "attention":
        b, f = _attention_work(case["nq"], case["nkv"], case["d"], case["prefix"], case["suffix"])
        return {"bytes": b, "flops": f}
    if kind == "ingest":
        return {"bytes": 2 * case["prefix"] * 4 * case["nkv"] * case["d"], "flops": 0}
    if kind == "chunk_objects":
        tokens = case["prefix"] + case["suffix"] + (case["suffix"] // case["chunk"]) * case["chunk"]
        return {"bytes": 2 * tokens * case["layers"] * 4 * case["nkv"] * case["d"], "flops": 0}
    if kind == "rest_of_layer":
        T, H, F, n_qkv = case["tokens"], case["nq"] * case["d"], case["ffn"], (case["nq"] + 2 * case["nkv"]) * case["d"]
        params = H * H + H * 2 * F + F * H + H * n_qkv
        return {"bytes": 2 * (params + T * (H + H + 2 * F + F + H + n_qkv)), "flops": 2 * T * params}
    b = f = 0
    row = 4 * case["nkv"] * case["d"]
    for t in (int(x) for x in case["prefixes"].split()):
        ab, af = _attention_work(case["nq"], case["nkv"], case["d"], t, case["suffix"])
        # payload read, pool written (then read by the attention), suffix appended
        b += ab + 2 * t * row + (case["suffix"] * row if case["append"] else 0)
        f += af
    return {"bytes": b * case["layers"], "flops": f * case["layers"]}


def tolerance(case):
    kind = case["kind"]
    if kind in ("ingest", "chunk_objects"):
        return "exact"
    if kind == "rest_of_layer":
        # four chained GEMMs, each stage rounded to bfloat16
        return {"rel": 1e-2, "max": 0.1}
    # bfloat16 output, probabilities rounded to bfloat16 before the PV product
    return {"rel": 1e-2, "max": 0.1, "differ": 0.0}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _exact_attention(q, K, V):
    """q [ts][nq][d]; K, V [tp + ts][nkv][d]; causal within the last ts keys."""
    ts, nq, d = q.shape
    n, nkv, _ = K.shape
    grp = nq // nkv
    out = torch.empty(ts, nq, d, dtype=torch.float64, device=q.device)
    at = torch.arange(n, device=q.device)
    for h in range(nkv):
        k, v = K[:, h].double(), V[:, h].double()
        step = max(1, (1 << 27) // (n * grp))
        for i in range(0, ts, step):
            qs = q[i:i + step, h * grp:(h + 1) * grp].double()
            m = qs.shape[0]
            s = (qs.reshape(m * grp, d) @ k.t()).reshape(m, grp, n) / math.sqrt(d)
            seen = at[None, :] <= (n - ts + i + torch.arange(m, device=q.device))[:, None]
            s = s.masked_fill(~seen[:, None, :], float("-inf"))
            p = torch.softmax(s, dim=-1)
            out[i:i + m, h * grp:(h + 1) * grp] = (p.reshape(m * grp, n) @ v).reshape(m, grp, d)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "attention":
        lay, pool, table, q, k, v = _attention(case, seed)
        kv = pool.view(2, lay.num_pages, lay.num_kv_heads, PAGE, lay.head_dim)[:, table.long()]
        kv = kv.permute(0, 1, 3, 2, 4).reshape(2, -1, lay.num_kv_heads, lay.head_dim)[:, :case["prefix"]]
        return _exact_attention(q, torch.cat([kv[0], k]), torch.cat([kv[1], v]))
    if kind == "rest_of_layer":
        x, (w_o, w_gu, w_down, w_qkv) = _layer(case, seed)
        F = case["ffn"]
        o = x.double() @ w_o[0].double()
        gu = o @ w_gu[0].double()
        act = gu[:, :F] * torch.sigmoid(gu[:, :F]) * gu[:, F:]
        h = act @ w_down[0].double()
        return [o, gu, act, h, h @ w_qkv[0].double()]
    if kind == "pipeline":
        lay, tables, tps, reqs = _pipeline(case, seed)
        outs = []
        for t, (kv, q, k, v) in zip(tps, reqs):
            rows = kv.permute(0, 2, 1, 3, 4, 5).reshape(lay.num_layers, 2, t, lay.num_kv_heads, lay.head_dim)
            outs.append(torch.stack([_exact_attention(q[i], torch.cat([rows[i, 0], k[i]]),
                                                      torch.cat([rows[i, 1], v[i]])) for i in range(lay.num_layers)]))
        return {"out": outs, "pool": None}
    return None     # bytes moved as they are: nothing is computed


if __name__ == "__main__":
    for c in listed() + [draw(random.Random(s)) for s in range(8)]:
        print(c, work(c))
