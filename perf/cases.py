"""The calls whose speed users of this library feel, as measurable cases.

Two kinds of work:

prefill  one request: the whole prefix, block by block through every layer (attention over cache
         and block, scores, select, merge, compaction), starting from an empty cache.  Three ways to
         drive it, as in runtime.py and include/kvp.h:
           block      runtime.Prefill: every layer's block in one call (`overlap`: compactions on a second stream)
           layerwise  runtime.LayerwisePrefill: a model's order, one call per layer, then one for the stack
           calls      Cache.prefill_chunk and Cache.compact per layer, one scratch set
         scored by the block's own queries ("own"), by `n_obs` proxy queries of the prompt ("proxy")
         or by the keys alone ("keydiff").
decode   one generated token through every layer over a compressed cache (`static`: the entry point
         that borrows no scratch memory).

A prefix is one image (`planes` tiles) or one video (`planes` frames, `temporal`) of grid_h x grid_w
patch tokens per plane, followed by `text` tokens.  `chunk` and `budget` are the block size b and the
budget M of the method.
"""
import math

import torch

import paper_2604_16734_amd as kvp

BF16 = torch.bfloat16


def _prefill(name, driver, scoring, layers, hq, hkv, d, chunk, budget, grid_h, grid_w, planes, temporal, text,
             merge=True, sets=1, overlap=False, n_obs=0):
    case = dict(kind="prefill", driver=driver, scoring=scoring, layers=layers, hq=hq, hkv=hkv, d=d, chunk=chunk,
                budget=budget, grid_h=grid_h, grid_w=grid_w, planes=planes, temporal=temporal, text=text, merge=merge,
                sets=sets, overlap=overlap, n_obs=n_obs)
    return dict(case, name=name) if name else case


def _decode(name, layers, hq, hkv, d, count, tail, static=False):
    case = dict(kind="decode", layers=layers, hq=hq, hkv=hkv, d=d, count=count, tail=tail, static=static)
    return dict(case, name=name) if name else case


# The five workloads of kvp_workload/configs.py: (layers, query heads, KV heads, head dim, b, M, grid, planes, temporal, text)
TINY = (1, 4, 4, 64, 64, 128, 24, 24, 1, False, 32)
SINGLE_IMAGE = (4, 32, 32, 128, 128, 256, 24, 24, 1, False, 64)
TILED_IMAGE = (8, 28, 4, 128, 256, 512, 24, 24, 5, False, 128)
VIDEO = (16, 28, 4, 128, 512, 1024, 14, 14, 32, True, 128)
LONG_VIDEO = (32, 32, 8, 128, 1024, 2048, 16, 16, 64, True, 256)


def listed():
    return [
        # the smallest request: ten blocks of 64 tokens, all launches and latency
        _prefill("tiny block", "block", "own", *TINY),
        # one image through a few layers in a model's order: small blocks, every head its own KV head
        _prefill("single_image layerwise", "layerwise", "own", *SINGLE_IMAGE, sets=4),
        # an image cut into tiles, all layers of a block in one call
        _prefill("tiled_image block", "block", "own", *TILED_IMAGE, sets=8),
        # the same image through the two per-layer calls and nothing else, scored by the keys, evictions only
        _prefill("tiled_image calls keydiff", "calls", "keydiff", *TILED_IMAGE, merge=False),
        # a short video in a model's order
        _prefill("video layerwise", "layerwise", "own", *VIDEO, sets=16),
        # the same video, compactions on a second stream, scored by the prompt's 128 tokens
        _prefill("video overlap proxy", "block", "proxy", *VIDEO, sets=16, overlap=True, n_obs=128),
        # a long video, the benchmark's shape and launch order
        _prefill("long_video block", "block", "own", *LONG_VIDEO, sets=16),
        # the same video in a model's order, scored by 64 proxy queries
        _prefill("long_video layerwise proxy", "layerwise", "proxy", *LONG_VIDEO, sets=32, n_obs=64),
        # nothing is a multiple of anything: head dimension 64, odd block, budget, grid and text lengths
        _prefill("ragged layerwise", "layerwise", "own", 24, 16, 4, 64, 333, 1111, 13, 19, 37, True, 101, merge=False, sets=24),
        # generation after a single image, after a tiled image (static scratch) and after a long video
        _decode("decode single_image", 4, 32, 32, 128, 256, 9),
        _decode("decode tiled_image static", 8, 28, 4, 128, 512, 41, static=True),
        _decode("decode long_video", 32, 32, 8, 128, 2048, 128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


HEADS = [(4, 4), (32, 32), (28, 4), (32, 8), (16, 4), (8, 2), (6, 2)]


def draw(rng):
    most = work(_prefill(None, "block", "own", *LONG_VIDEO))
    while True:
        layers = _log_int(rng, 1, 32)
        hq, hkv = rng.choice(HEADS)
        d = rng.choice([64, 128, 128])
        if rng.random() < 0.25:
            case = _decode(None, layers, hq, hkv, d, _log_int(rng, 1, 6000), _log_int(rng, 1, 500), rng.random() < 0.3)
        else:
            chunk = _log_int(rng, 48, 1536)
            budget = _log_int(rng, 96, 4096)
            temporal = rng.random() < 0.5
            driver = rng.choice(["block", "block", "layerwise", "layerwise", "calls"])
            sets = {"block": rng.randint(1, min(layers, 16)), "layerwise": layers, "calls": 1}[driver]
            scoring = rng.choice(["own", "own", "own", "proxy", "keydiff"])
            case = _prefill(None, driver, scoring, layers, hq, hkv, d, chunk, budget, rng.randint(7, 28), rng.randint(7, 28),
                            _log_int(rng, 1, 96), temporal, _log_int(rng, 16, 300), rng.random() < 0.7, sets,
                            driver == "block" and sets >= 2 and rng.random() < 0.25,
                            min(chunk, _log_int(rng, 8, 256)) if scoring == "proxy" else 0)
            if not budget <= _tokens(case) <= 24000 or _tokens(case) > 120 * chunk:
                continue
        w = work(case)
        if w["flops"] <= 0.8 * most["flops"] and w["bytes"] <= most["bytes"]:
            return case


def _tokens(case):
    return case["grid_h"] * case["grid_w"] * case["planes"] + case["text"]


def _blocks(case):
    n, b = _tokens(case), case["chunk"]
    return [(t, min(b, n - t)) for t in range(0, n, b)]


def _grid_rows(case, gen):
    """Keys or values of the visual tokens of one layer: smooth fields over the patch grid (one per tile, or
    one for all frames with a slowly drifting offset) plus a little noise, as kvp_workload/generate.py draws them."""
    gh, gw, planes, hkv, d = (case[k] for k in ("grid_h", "grid_w", "planes", "hkv", "d"))
    units = 1 if case["temporal"] else planes
    dev = gen.device

    def uniform(hi):
        return hi * torch.rand((units, 1, 1, hkv, d, 4), generator=gen, device=dev)

    y = (torch.arange(gh, device=dev) / gh).view(1, gh, 1, 1, 1, 1)
    x = (torch.arange(gw, device=dev) / gw).view(1, 1, gw, 1, 1, 1)
    rows = torch.sin(2 * math.pi * (uniform(2.0) * y + uniform(2.0) * x) + uniform(2 * math.pi)).sum(-1) * 0.5 ** 0.5
    if case["temporal"]:
        drift = 0.5 * torch.randn((planes, hkv, d), generator=gen, device=dev)
        for i in range(1, planes):
            drift[i] = 0.9 * drift[i - 1] + (1 - 0.9 ** 2) ** 0.5 * drift[i]
        rows = rows + drift.view(planes, 1, 1, hkv, d)
    rows = rows.reshape(planes * gh * gw, hkv, d)
    return rows + 0.1 * torch.randn(rows.shape, generator=gen, device=dev)


def _over_layers(tensors):
    """One tensor over the equally spaced views of consecutive layers."""
    first = tensors[0]
    step = (tensors[1].data_ptr() - first.data_ptr()) // first.element_size() if len(tensors) > 1 else first.numel()
    return torch.as_strided(first, (len(tensors),) + tuple(first.shape), (step,) + tuple(first.stride()))


def _prepare_prefill(case, gen):
    layers, hq, hkv, d, n = case["layers"], case["hq"], case["hkv"], case["d"], _tokens(case)
    dev, n_vis = gen.device, n - case["text"]
    segments = [kvp.KvpSegment(0, n_vis, kvp.KVP_VISUAL, case["grid_h"], case["grid_w"], case["planes"], int(case["temporal"])),
                kvp.KvpSegment(n_vis, case["text"], kvp.KVP_TEXT, 0, 0, 0, 0)]
    cache = kvp.Cache(layers, hq, hkv, d, case["budget"], case["chunk"], segments, merge=case["merge"], scratch_sets=case["sets"])
    q = torch.randn((layers, n, hq, d), generator=gen, device=dev, dtype=BF16)
    k = torch.randn((layers, n, hkv, d), generator=gen, device=dev, dtype=BF16)
    v = torch.randn((layers, n, hkv, d), generator=gen, device=dev, dtype=BF16)
    for layer in range(layers):
        k[layer, :n_vis] = _grid_rows(case, gen)
        v[layer, :n_vis] = _grid_rows(case, gen)
    obs = None
    if case["scoring"] == "proxy":
        obs = list(torch.randn((layers, case["n_obs"], hq, d), generator=gen, device=dev, dtype=BF16))
    out = torch.empty_like(q)
    views = [cache.decode_ready(layer) for layer in range(layers)]
    state = dict(
        case=case, cache=cache, obs=obs, out=out,
        blocks=[(t, [(q[i, t:t + m], k[i, t:t + m], v[i, t:t + m], out[i, t:t + m]) for i in range(layers)])
                for t, m in _blocks(case)],
        # rows are copied or averaged once, in a fixed order: they are compared as bits
        cached=dict(k=_over_layers([w[0].view(torch.int16) for w in views]), v=_over_layers([w[1].view(torch.int16) for w in views]),
                    token=_over_layers([w[2] for w in views]), weight=_over_layers([w[3].view(torch.int32) for w in views])))
    if case["driver"] == "block":
        state["prefill"] = kvp.Prefill(cache, layers, overlap=case["overlap"])
    elif case["driver"] == "layerwise":
        state["prefill"] = kvp.LayerwisePrefill(cache, layers)
    return state


def _prepare_decode(case, gen):
    layers, hq, hkv, d, count, tail = (case[k] for k in ("layers", "hq", "hkv", "d", "count", "tail"))
    dev = gen.device
    cache = kvp.Cache(layers, hq, hkv, d, count, min(count, 1024), [kvp.KvpSegment(0, 2 * count, kvp.KVP_TEXT, 0, 0, 0, 0)])
    for layer in range(layers):
        k, v, token, weight, _, _ = cache.decode_ready(layer)
        k.copy_(torch.randn(k.shape, generator=gen, device=dev))
        v.copy_(torch.randn(v.shape, generator=gen, device=dev))
        token.copy_(torch.arange(count, device=dev, dtype=torch.int32).expand(hkv, count))
        weight.fill_(1.0)
        cache.set_state(layer, count, 2 * count)
    draw_ = lambda *shape: torch.randn(shape, generator=gen, device=dev, dtype=BF16)
    out = torch.empty((layers, hq, d), device=dev, dtype=BF16)
    return dict(case=case, cache=cache, out=out,
                token=list(zip(draw_(layers, hq, d), draw_(layers, tail, hkv, d), draw_(layers, tail, hkv, d), out)))


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return _prepare_prefill(case, gen) if case["kind"] == "prefill" else _prepare_decode(case, gen)


def run(state):
    case, cache = state["case"], state["cache"]
    if case["kind"] == "decode":
        step = cache.decode_step_static if case["static"] else cache.decode_step
        for layer, (q, k, v, out) in enumerate(state["token"]):
            step(layer, q, k, v, out)
        return state["out"]
    layers, scoring, obs = case["layers"], case["scoring"], state["obs"]
    for layer in range(layers):
        cache.set_state(layer, 0, 0)          # a new request: the cache is empty again
    if case["driver"] == "block":
        prefill = state["prefill"]
        for t, of in state["blocks"]:
            prefill.block(t, lambda i: of[i][:3], lambda i: of[i][3], obs.__getitem__ if obs else None, scoring == "keydiff")
        prefill.finish()
    elif case["driver"] == "layerwise":
        prefill = state["prefill"]
        for t, of in state["blocks"]:
            for layer, (q, k, v, out) in enumerate(of):
                prefill.layer(layer, t, q, k, v, out, obs[layer] if obs else None, scoring == "keydiff")
            prefill.end_block()
    else:
        for t, of in state["blocks"]:
            for layer, (q, k, v, out) in enumerate(of):
                if scoring == "keydiff":
                    cache.prefill_chunk_keydiff(layer, t, q, k, v, out)
                elif scoring == "proxy":
                    cache.prefill_chunk_proxy(layer, t, q, k, v, obs[layer], out)
                else:
                    cache.prefill_chunk(layer, t, q, k, v, out)
                cache.compact(layer)
    return dict(state["cached"], out=state["out"])


def work(case):
    """Every input read once, every output written once; the products of attention (and of the proxy queries with
    the candidates of a block that evicts), but no second product for the block's own scores: their logits are
    those of the attention."""
    layers, hq, hkv, d = case["layers"], case["hq"], case["hkv"], case["d"]
    if case["kind"] == "decode":
        keys = case["count"] + case["tail"]
        return {"bytes": layers * (2 * hkv * keys * d + 2 * hq * d) * 2, "flops": layers * 4 * d * hq * keys}
    n, m = _tokens(case), case["budget"]
    flops, count = 0, 0
    for _, b in _blocks(case):
        flops += 4 * d * hq * (b * count + b * (b + 1) // 2)
        if count + b > m and case["scoring"] == "proxy":
            flops += 2 * d * hq * case["n_obs"] * (count + b)
        count = min(m, count + b)
    rows = 2 * n * hq + 2 * n * hkv + case["n_obs"] * hq + 2 * m * hkv
    return {"bytes": layers * (rows * d * 2 + m * hkv * 8), "flops": layers * flops}


def tolerance(case):
    """Attention outputs are bf16 from fp32 sums of bf16 products.  Selected rows are bits, but which of two
    candidates with scores equal to the last fp32 digits is kept (and with it the slots and merges after it)
    may differ: a small share of the slots, and what such a swap does to single elements of later outputs (two orders
    of summing the scores, tried over these ranges: 0.3 % of the slots, 0.5 of the root mean square in one element)."""
    if case["kind"] == "decode":
        return {"rel": 1e-2, "max": 5e-2}
    return {"rel": 1e-2, "max": 9e-1, "differ": 1e-2}
