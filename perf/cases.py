"""The work this library is used for, as measurable cases.

Two kinds, both through the package's public calls:

  evict   laq_evict: score every key of a cache with the observation window's queries, keep the best
          `budget` rows per KV head, gather their K and V rows (the low-budget first eviction and the
          re-eviction of the method, one layer at a time or all layers of a batch in one call)
  decode  laq_decode_attention over the compacted cache, one new token per (sequence, layer); with
          `store`, also laq_qcache_store of the step's queries, as every lookahead step does

Fields of a case: n = (sequence, layer) instances of the call; heads, kv_heads, d, L, W, dtype, pool,
pool_mode as in the library's shape; budget_hi / budget_lo = rows kept per KV head, falling linearly over
the instances; window = trailing | joined (up to 8 local queries, the others generated after the
prompt) | lookahead (all of them after the prompt, nothing kept); layout = dense | token_major | paged (blocks of
`block` rows behind a shuffled table); keys = heavy | clusters | tails (the structure of the inputs);
own = the caller keeps output buffers and workspace from call to call (False: the package makes them).
"""
import math

import torch

import paper_2505_20334_amd as laq

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
# K' and V' are copies of rows: they are handed back as the whole numbers of their bits
BITS = {torch.bfloat16: torch.int16, torch.float32: torch.int32}


def _evict(name=None, **kw):
    case = dict(kind="evict", n=1, heads=32, kv_heads=8, d=128, L=4096, W=8, dtype="bf16", pool=7, pool_mode="max",
                budget_hi=128, budget_lo=128, window="trailing", layout="dense", block=0, keys="heavy", own=False)
    case.update(kw)
    if name:
        case["name"] = name
    return case


def _decode(name=None, **kw):
    case = dict(kind="decode", n=1, heads=32, kv_heads=8, d=128, L=16384, W=8, dtype="bf16", budget_hi=512,
                budget_lo=512, store=False, own=False)
    case.update(kw)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest call: a fp32 toy model, one layer of 512 keys; launches and host work are all of it
        _evict("evict-tiny-f32", heads=4, kv_heads=2, d=64, L=512, dtype="f32", budget_hi=64, budget_lo=64),
        # one layer of an 8B-shaped model with a 4k prompt, evicted as soon as the layer is prefilled
        _evict("evict-layer-4k", L=4096),
        # the method's main setting (8 local + 8 lookahead queries) on one layer of a long prompt of no
        # round length, in a serving loop that keeps its buffers
        _evict("evict-layer-joined-30k", L=30011, W=16, window="joined", budget_hi=1024, budget_lo=1024, own=True),
        # the low-budget first eviction: average pool, 8 local queries, the cache as a token-major model
        # stores it
        _evict("evict-first-stage-8k", n=32, L=8001, W=8, pool_mode="avg", layout="token_major"),
        # re-eviction of all layers of a 16k prompt
        _evict("evict-32layer-16k", n=32, L=16384, W=16, budget_hi=512, budget_lo=512),
        # all layers of a 32k prompt, 32 lookahead queries, pyramid budgets (the benchmark's headline)
        _evict("evict-32layer-32k", n=32, L=32768, W=32, budget_hi=2048, budget_lo=128, keys="clusters", own=True),
        # a serving engine's paged cache, seven query heads per KV head, joined window, ragged length
        _evict("evict-paged-gqa7-20k", n=28, heads=28, kv_heads=4, L=20123, W=16, window="joined", layout="paged",
               block=256, budget_hi=512, budget_lo=512),
        # the largest call: eight 32k prompts, all layers
        _evict("evict-batch8-32k", n=256, L=32768, W=16, budget_hi=256, budget_lo=256, keys="tails", own=True),
        # fp32 caches of a few layers (quality studies compare with full precision)
        _evict("evict-8layer-8k-f32", n=8, L=8191, W=16, dtype="f32", budget_hi=256, budget_lo=256),
        # one lookahead step of one layer: a single token over a small cache, its queries captured
        _decode("decode-layer-lookahead", n=1, budget_hi=512, budget_lo=512, store=True),
        # one token over the pyramid cache of all layers
        _decode("decode-32layer-pyramid", n=32, L=32768, budget_hi=2048, budget_lo=128, own=True),
        # eight sequences, all layers, small caches: as many short caches as the largest eviction leaves
        _decode("decode-batch8-256", n=256, L=32768, budget_hi=256, budget_lo=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    heads, kv_heads = rng.choice([(32, 8), (32, 8), (32, 8), (28, 4), (16, 8), (32, 32), (8, 1)])
    d = rng.choices([128, 64, 96, 256], [60, 24, 8, 8])[0]
    dtype = rng.choices(["bf16", "f32"], [85, 15])[0]
    eb = 2 if dtype == "bf16" else 4
    n = _log_int(rng, 1, 256)
    hi = _log_int(rng, 64, 2048)
    lo = max(64, int(hi * rng.choice([1.0, 1.0, 0.5, 0.0625])))
    own = rng.random() < 0.4
    if rng.random() < 0.3:
        n = min(n, max(1, (2 << 30) // (2 * kv_heads * hi * d * eb)))
        return _decode(n=n, heads=heads, kv_heads=kv_heads, d=d, L=_log_int(rng, hi, 32768), W=8, dtype=dtype,
                       budget_hi=hi, budget_lo=lo, store=rng.random() < 0.5, own=own)
    L = _log_int(rng, 320, 32768)
    if rng.random() < 0.3:
        L = max(512, L // 256 * 256)
    # the keys of the call stay below half of the largest listed one's (an eighth of that outside the usual
    # head sizes and for fp32)
    most = (8 << 30) if dtype == "bf16" and d in (64, 128) else (512 << 20)
    n = min(n, max(1, most // (kv_heads * L * d * eb)))
    W = rng.choice([8, 8, 16, 16, 32])
    window = rng.choice(["trailing", "joined", "lookahead"])
    layout = rng.choices(["dense", "token_major", "paged"], [60, 20, 20])[0]
    return _evict(n=n, heads=heads, kv_heads=kv_heads, d=d, L=L, W=W, dtype=dtype, pool=rng.choice([7, 7, 7, 5, 13]),
                  pool_mode=rng.choices(["max", "avg"], [80, 20])[0], budget_hi=min(hi, L), budget_lo=min(lo, L),
                  window=window, layout=layout, block=rng.choice([256, 512]) if layout == "paged" else 0,
                  keys=rng.choice(["heavy", "clusters", "tails"]), own=own)


def _budgets(case):
    n, hi, lo = case["n"], case["budget_hi"], case["budget_lo"]
    return [hi - (hi - lo) * i // max(1, n - 1) for i in range(n)]


def _window(case):
    """(q_pos, keep) of the call."""
    L, W = case["L"], case["W"]
    if case["window"] == "trailing":
        return None, None
    local = min(8, W // 2) if case["window"] == "joined" else 0
    return [L - local + i for i in range(local)] + [L + i for i in range(W - local)], local


def _key_rows(case, q, gen):
    """Keys of the instances of q [m, heads, W, d]: [m, kv_heads, L, d]."""
    m, L, d, H = q.shape[0], case["L"], case["d"], case["kv_heads"]
    dt, dev = q.dtype, q.device
    k = torch.randn(m, H, L, d, generator=gen, device=dev, dtype=dt)
    if case["keys"] == "clusters":
        # keys of one topic lie together: 64 centres per head
        centres = torch.randn(m, H, 64, d, generator=gen, device=dev, dtype=dt)
        which = torch.randint(0, 64, (m, H, L), generator=gen, device=dev)
        k.mul_(0.5).add_(torch.gather(centres, 2, which.unsqueeze(-1).expand(m, H, L, d)))
    elif case["keys"] == "heavy":
        # a few keys the window looks for, all over the prompt, and the attention sink at its start
        look = torch.nn.functional.normalize(q.float().reshape(m, H, -1, d).mean(2), dim=-1)
        count = max(4, L // 128)
        stride = L // count
        pos = torch.arange(count, device=dev) * stride + torch.randint(0, stride, (m, H, count), generator=gen, device=dev)
        amp = 2.0 + 4.0 * torch.rand(m, H, count, 1, generator=gen, device=dev)
        rows = amp * look.unsqueeze(2) + torch.randn(m, H, count, d, generator=gen, device=dev)
        k.scatter_(2, pos.unsqueeze(-1).expand(m, H, count, d), rows.to(dt))
        k[:, :, :4] = (8.0 * look.unsqueeze(2) + torch.randn(m, H, 4, d, generator=gen, device=dev)).to(dt)
    return k


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + 13)
    dt, n, Hq, H, d, L, W = DTYPES[case["dtype"]], case["n"], case["heads"], case["kv_heads"], case["d"], case["L"], case["W"]
    budgets = _budgets(case)
    rows = sum(H * min(b, L) for b in budgets)
    state = {"kind": case["kind"], "budgets": budgets, "bits": BITS[dt]}
    if case["kind"] == "decode":
        q = torch.randn(n, Hq, d, generator=gen, device=dev, dtype=dt)
        kc = torch.randn(rows, d, generator=gen, device=dev, dtype=dt)
        vc = torch.randn(rows, d, generator=gen, device=dev, dtype=dt)
        state.update(args=(q, kc, vc, budgets, H, L), kw={}, q_cache=None)
        if case["store"]:
            state["q_cache"] = torch.randn(n, Hq, W, d, generator=gen, device=dev, dtype=dt)
            state["slot"] = int(seed) % W
        if case["own"]:
            need = laq.laq_decode_workspace_bytes(n, Hq, H, d, L, dt, budgets)
            state["kw"] = {"out": torch.empty(n, Hq, d, device=dev), "ws": torch.empty(max(16, need), dtype=torch.uint8, device=dev)}
        return state

    q = torch.randn(n, Hq, W, d, generator=gen, device=dev)
    if case["keys"] == "tails":
        # heavy-tailed query norms (Student-t, three degrees of freedom)
        t = torch.randn(n, Hq, W, 4, generator=gen, device=dev)
        q *= (t[..., :1] / (t[..., 1:].square().sum(-1, keepdim=True) / 3.0).sqrt()).abs()
    q = q.to(dt)
    table = None
    br, per = case["block"], 0
    if case["layout"] == "paged":
        per = -(-L // br)
        table = torch.randperm(n * per, generator=gen, device=dev).reshape(n, per).int()
        k, v = (torch.zeros(n * per, H, br, d, device=dev, dtype=dt) for _ in range(2))
    elif case["layout"] == "token_major":
        k, v = (torch.empty(n, L, H, d, device=dev, dtype=dt).permute(0, 2, 1, 3) for _ in range(2))
    else:
        k, v = (torch.empty(n, H, L, d, device=dev, dtype=dt) for _ in range(2))
    step = max(1, (1 << 28) // (H * L * d))
    for i in range(0, n, step):
        qi = q[i:i + step]
        m = qi.shape[0]
        for dst, src in ((k, _key_rows(case, qi, gen)), (v, torch.randn(m, H, L, d, generator=gen, device=dev, dtype=dt))):
            if table is not None:
                src = torch.nn.functional.pad(src, (0, 0, 0, per * br - L)).reshape(m, H, per, br, d).transpose(1, 2)
                dst[table[i:i + m].long()] = src
            else:
                dst[i:i + m] = src
    q_pos, keep = _window(case)
    kw = {"pool_mode": case["pool_mode"], "q_pos": q_pos, "keep": keep}
    if table is not None:
        kw.update(block_table=table, L=L)
    if case["own"]:
        kw.update(scores=torch.empty(n, H, L, device=dev), idx=torch.empty(rows, dtype=torch.int32, device=dev),
                  k_out=torch.empty(rows, d, dtype=dt, device=dev), v_out=torch.empty(rows, d, dtype=dt, device=dev),
                  ws=torch.empty(laq.laq_workspace_bytes(n, Hq, H, d, L, W, dt, q_pos, keep), dtype=torch.uint8, device=dev))
    state.update(args=(q, k, v, budgets, case["pool"]), kw=kw)
    return state


def run(state):
    if state["kind"] == "decode":
        out = {"out": laq.laq_decode_attention(*state["args"], **state["kw"])}
        if state["q_cache"] is not None:
            out["q_cache"] = laq.laq_qcache_store(state["q_cache"], state["args"][0], state["slot"])
        return out
    scores, idx, k_out, v_out = laq.laq_evict(*state["args"], **state["kw"])
    return {"scores": scores, "idx": idx, "k": k_out.view(state["bits"]), "v": v_out.view(state["bits"])}


def work(case):
    eb = 2 if case["dtype"] == "bf16" else 4
    n, Hq, H, d, L, W = case["n"], case["heads"], case["kv_heads"], case["d"], case["L"], case["W"]
    rows = sum(H * min(b, L) for b in _budgets(case))
    if case["kind"] == "decode":
        # q, K' and V' read, the output written; the step's queries written to the Q-cache
        stored = n * Hq * d * eb if case["store"] else 0
        return {"bytes": n * Hq * d * (eb + 4) + 2 * rows * d * eb + stored, "flops": 4 * rows * (Hq // H) * d}
    # q and K read once, the scores and the list written, the retained V rows read, K' and V' written
    return {"bytes": (n * Hq * W + n * H * L + 3 * rows) * d * eb + 4 * n * H * L + 4 * rows,
            "flops": 2 * n * Hq * W * L * d}


def tolerance(case):
    # scores and attention: fp32 sums of exponentials of fp32 dot products (of bf16 inputs: longer exponents,
    # whose absolute rounding the exponential makes relative).  Lists and the rows they name: two scores next
    # to a cut that are equal to within that rounding may change places, which moves the entries between them.
    return {"rel": 1e-4 if case["dtype"] == "bf16" else 2e-5, "differ": 0.01}
