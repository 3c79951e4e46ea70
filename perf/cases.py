"""Timed cases of the decode-step path: whole layer-steps (`ess_decode_step`, with `ess_append` where a program
appends after each step) and the single stages a program can call by themselves.

Indexer and attention sizes are those of bench.py (64 indexer heads x 128 e4m3, top-2048, 128 attention heads x 576),
batches and contexts those of its workloads and of the paper's tables (batches 13, 32, 40, 64, 128 at 32K and 128K
context), with smaller, odd and ragged ones between.

Inputs.  Indexer queries and keys are integers in [-8, 8] stored as e4m3 and head weights are sixteenths, so that a
score is one number whatever the order of its sum, and a selection one set.  Successive decode steps of a sequence
use related queries: element d of the query takes one of two values and changes between them once in 32 steps, at a
step of its own, over a ring of 64 steps.  Real selections made with such queries share 70-80 % of their entries from
step to step (the Intra-Layer Similarity that the paper measures) and miss 150-300 of 2048 entries at slot pools of 10 to 25 %
of the context.  An offloaded state has run once round the ring, so its pool is in its steady state.

`exact` computes in float64 with torch alone and shares nothing with the library but the byte layouts.
"""
import math

import torch

from paper_2512_10576_amd import binding as bnd

DEV = "cuda"
RING = 64            # decode steps after which the queries repeat
ATTN_SETS = 4        # attention queries in hand, used in turn
SCALE = 576 ** -0.5
PAGE = 64
LARGEST_POOL = 128 * 131072 * 656    # bytes of Latent-Cache of the largest case


# ------------------------------------------------------------------ the cases

def _step(name, B, L, lo, hi=None, T=1, fmt="bf16", slots=0, paged=False, append=False, Hi=64, Di=128, k=2048, H=128):
    return dict(name=name, kind="step", B=B, T=T, L=L, lo=lo, hi=hi or L, fmt=fmt, slots=slots, paged=paged, append=append,
                Hi=Hi, Di=Di, k=k, H=H)


def listed():
    return [
        # one user with a short conversation: launches and latency
        _step("step-1x8k", 1, 8192, 8000),
        # a few users with long documents, resident
        _step("step-4x128k", 4, 131072, 100000),
        # the resident 32K workload of bench.py
        _step("step-32x32k", 32, 32768, 32768),
        # the same context offloaded to host memory, a quarter of it in slots
        _step("step-64x32k-offload", 64, 32768, 32768, slots=8192),
        # the default workload of bench.py: ragged 128K contexts, a tenth of them in slots
        _step("step-64x128k-offload", 64, 131072, 98304, slots=13108),
        # the multi-token workload of bench.py with quantised entries, one layer: the largest call
        _step("step-128x128k-mtp2-fp8", 128, 131072, 131072, T=2, fmt="fp8", slots=13108),
        # a server's inner loop: paged keys, two draft tokens, odd batch, the new entries appended after each step
        _step("serve-23x48k-mtp2-paged", 23, 49152, 24000, 40000, T=2, fmt="fp8", slots=9001, paged=True, append=True),
        # index score by itself, activations with a normal distribution and signed head weights (the paper's largest
        # resident batch at 128K)
        dict(name="score-13x128k", kind="score", B=13, T=1, L=131072, Hi=64, Di=128),
        # selection by itself over paged keys (the paper's offloaded batch at 128K)
        dict(name="select-40x100k-paged", kind="select", B=40, T=1, L=102400, lo=60000, paged=True, Hi=64, Di=128, k=2048),
        # look-up, LRU update and fetch with the selected rows handed to a program's own attention
        dict(name="gather-32x64k", kind="gather", B=32, T=1, L=65536, slots=6554, k=2048, fmt="bf16"),
        # attention of a tensor-parallel shard: 16 of 128 heads, two tokens
        dict(name="mla-16x2-16heads", kind="mla", B=16, T=2, S=8192, k=2048, H=16, fmt="bf16", ragged=False),
        # attention over quantised entries, lists of uneven length
        dict(name="mla-48x2-fp8-ragged", kind="mla", B=48, T=2, S=13108, k=2048, H=128, fmt="fp8", ragged=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: batches 1-128, contexts 1K-128K, one or two query tokens (now and then four),
    both entry formats, resident and offloaded, flat and paged keys."""
    kind = rng.choice(["step"] * 5 + ["score", "select", "gather", "mla", "mla"])
    B = _log(rng, 1, 128)
    T = rng.choice([1, 1, 1, 2, 2, 4])
    L = _log(rng, 1024, 131072)
    fmt = rng.choice(["bf16", "fp8"])
    stride = 1152 if fmt == "bf16" else 656
    k = rng.choice([2048, 2048, 2048, 2048, 1024, 513])
    H = rng.choice([128, 128, 128, 64, 16, 40])
    Hi = rng.choice([64, 64, 64, 32])
    B = max(1, min(B, LARGEST_POOL // (L * stride), 256 // T))
    if kind == "score":
        return dict(kind=kind, B=B, T=1, L=L, Hi=Hi, Di=rng.choice([128, 128, 64]))
    if kind == "select":
        paged = rng.random() < 0.5
        L = max(PAGE, L // PAGE * PAGE) if paged else L
        return dict(kind=kind, B=B, T=min(T, 2), L=L, lo=max(1, int(L * rng.uniform(0.5, 1.0))), paged=paged, Hi=Hi, Di=128, k=k)
    if kind == "mla":
        return dict(kind=kind, B=B, T=T, S=max(_log(rng, 2048, 32768), k), k=k, H=H, fmt=fmt, ragged=rng.random() < 0.5)
    if kind == "gather":
        T = min(T, 2)
        L = max(L, 4 * T * k)
        B = max(1, min(B, LARGEST_POOL // (L * stride)))
        return dict(kind=kind, B=B, T=T, L=L, slots=max(T * k + rng.randrange(64), int(L * rng.uniform(0.1, 0.3))), k=k, fmt=fmt)
    paged, append, offload = rng.random() < 0.4, rng.random() < 0.3, rng.random() < 0.6
    if paged:
        L = max(PAGE, L // PAGE * PAGE)
    slots = 0
    if offload:
        L = max(L, 4 * T * k // PAGE * PAGE + PAGE)
        B = max(1, min(B, LARGEST_POOL // (L * stride)))
        slots = max(T * k + rng.randrange(64), int(L * rng.uniform(0.1, 0.3)))
    hi = int(L * 0.75) if append else L
    c = _step("", B, L, max(1, int(hi * rng.uniform(0.6, 1.0))), hi, T, fmt, slots, paged, append, Hi, 128, k, H)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 64 + what)
    return g


def _e4m3(x):
    return x.to(torch.float32).to(torch.float8_e4m3fn).view(torch.uint8)


def _value(bytes_):
    """the numbers that e4m3 bytes stand for, in 64 bits"""
    return bytes_.view(torch.float8_e4m3fn).to(torch.float32).to(torch.float64)


def _stride(c):
    return 1152 if c["fmt"] == "bf16" else 656


def _entries(g, n, fmt):
    """n Latent-Cache entries with N(0,1) values, as bytes"""
    x = torch.randn((n, 576), generator=g, device=DEV)
    if fmt == "bf16":
        return x.to(torch.bfloat16).view(torch.uint8).view(n, 1152)
    lat = x[:, :512].view(n, 4, 128)
    scale = (lat.abs().amax(dim=-1) / 448.0).to(torch.bfloat16)
    rows = torch.zeros((n, 656), dtype=torch.uint8, device=DEV)
    rows[:, :512] = _e4m3((lat / scale.to(torch.float32).unsqueeze(-1)).clamp(-448.0, 448.0)).view(n, 512)
    rows[:, 512:520] = scale.view(torch.uint8).view(n, 8)
    rows[:, 520:648] = x[:, 512:].to(torch.bfloat16).view(torch.uint8).view(n, 128)
    return rows


def _entry_values(rows, fmt):
    """[n,576] in 64 bits"""
    if fmt == "bf16":
        return rows.view(torch.bfloat16).to(torch.float64)
    n = rows.shape[0]
    lat = _value(rows[:, :512].contiguous()).view(n, 4, 128)
    scale = rows[:, 512:520].contiguous().view(torch.bfloat16).to(torch.float64)
    rope = rows[:, 520:648].contiguous().view(torch.bfloat16).to(torch.float64)
    return torch.cat([(lat * scale.unsqueeze(-1)).view(n, 512), rope], dim=1)


def _lengths(c, seed):
    return torch.randint(c["lo"], c.get("hi", c["L"]) + 1, (c["B"],), generator=_gen(seed, 1), device=DEV, dtype=torch.int32)


def _integers(g, *shape):
    return torch.randint(-8, 9, shape, generator=g, device=DEV, dtype=torch.int8)


def _index_queries(c, seed):
    """(ring of queries [RING,B,T,Hi,Di] e4m3 bytes, head weights [B,T,Hi])"""
    g = _gen(seed, 2)
    shape = (c["B"], c["T"], c["Hi"], c["Di"])
    a, b = _integers(g, *shape), _integers(g, *shape)
    turn = torch.randint(0, RING, shape, generator=g, device=DEV, dtype=torch.int16)
    # the tokens of one step are close to each other, as those of successive steps are
    a, b, turn = (x[:, :1].expand(shape) for x in (a, b, turn))
    turn = turn + torch.arange(c["T"], device=DEV, dtype=torch.int16).view(1, -1, 1, 1)
    w = torch.randint(1, 9, shape[:3], generator=g, device=DEV).to(torch.float32) / 16
    return torch.stack([_e4m3(torch.where(torch.remainder(s - turn, RING) < RING // 2, a, b)) for s in range(RING)]), w


def _keys(c, seed, b):
    """index keys of sequence b: [L,Di] e4m3 bytes"""
    return _e4m3(_integers(_gen(seed, 1024 + b), c["L"], c["Di"]))


def _pages(c, seed):
    """(place of each page in the pool [B,L/64], scale of each key [B,L])"""
    g = _gen(seed, 3)
    n = c["L"] // PAGE
    place = torch.randperm(c["B"] * n, generator=g, device=DEV).to(torch.int32).view(c["B"], n).contiguous()
    return place, 0.5 + torch.rand((c["B"], c["L"]), generator=g, device=DEV, dtype=torch.float32)


def _key_store(c, seed):
    """(keys as the library takes them, block table or None)"""
    B, L, Di = c["B"], c["L"], c["Di"]
    if not c.get("paged"):
        keys = torch.empty((B, L, Di), dtype=torch.uint8, device=DEV)
        for b in range(B):
            keys[b] = _keys(c, seed, b)
        return keys, None
    place, scale = _pages(c, seed)
    pool = torch.empty((B * (L // PAGE), PAGE * (Di + 4)), dtype=torch.uint8, device=DEV)
    for b in range(B):
        at = place[b].long()
        pool[at, :PAGE * Di] = _keys(c, seed, b).view(-1, PAGE * Di)
        pool[at, PAGE * Di:] = scale[b].view(-1, PAGE).view(torch.uint8)
    return pool, place


def _attn_queries(c, seed, sets=ATTN_SETS):
    return torch.randn((sets, c["B"], c["T"], c["H"], 576), generator=_gen(seed, 4), device=DEV).to(torch.bfloat16)


def _latents(c, seed, b):
    return _entries(_gen(seed, 2048 + b), c["L"], c["fmt"])


def _new_entries(c, seed):
    """what the steps of the ring append: keys [RING,B,T,Di], scales [RING,B,T], entries [RING,B,T,stride]"""
    g = _gen(seed, 5)
    n = RING * c["B"] * c["T"]
    keys = _e4m3(_integers(g, n, c["Di"])).view(RING, c["B"], c["T"], c["Di"])
    scale = 0.5 + torch.rand((RING, c["B"], c["T"]), generator=g, device=DEV, dtype=torch.float32)
    return keys, scale, _entries(g, n, c["fmt"]).view(RING, c["B"], c["T"], _stride(c))


def _config(c, **kw):
    d = dict(max_batch=c["B"], max_q_tokens=c["T"], max_ctx=c.get("L", c.get("S")), idx_heads=c.get("Hi", 64), idx_dim=c.get("Di", 128),
             topk=c.get("k", 2048), attn_heads=c.get("H", 128),
             latent_fmt=bnd.ESS_FMT_FP8 if c.get("fmt") == "fp8" else bnd.ESS_FMT_BF16)
    d.update(kw)
    return bnd.make_config(**d)


def _host_pool(c, seed):
    pool = torch.empty((c["B"], c["L"], _stride(c)), dtype=torch.uint8, pin_memory=True)
    for b in range(c["B"]):
        pool[b].copy_(_latents(c, seed, b))
    return pool


# ------------------------------------------------------------------ states and passes

def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return globals()["_run_" + state["kind"]](state)


def _prepare_step(c, seed):
    B, T, L, k, H = c["B"], c["T"], c["L"], c["k"], c["H"]
    cfg = _config(c, slots_per_seq=c["slots"] or L, flags=bnd.ESS_FLAG_AUTO if c["slots"] else 0)
    s = dict(kind="step", case=c, step=0, ctx=bnd.Context(cfg))
    s["q"], s["w"] = _index_queries(c, seed)
    s["keys"], s["table"] = _key_store(c, seed)
    s["len"] = _lengths(c, seed)
    s["q_attn"] = _attn_queries(c, seed)
    if c["slots"]:
        s["cache"] = bnd.Cache.allocate(cfg, B, host_pool=_host_pool(c, seed))
    else:
        pool = torch.empty((B, L, _stride(c)), dtype=torch.uint8, device=DEV)
        for b in range(B):
            pool[b] = _latents(c, seed, b)
        s["cache"] = bnd.Cache.allocate(cfg, B, slot_pool=pool)
    s["ctx"].cache_reset(s["cache"], B)
    if c["append"]:
        s["new_key"], s["new_scale"], s["new_rows"] = _new_entries(c, seed)
        s["placed"] = torch.empty((B, T), dtype=torch.int32, device=DEV)
    s["idx"] = torch.empty((B, T, k), dtype=torch.int32, device=DEV)
    s["out"] = torch.empty((B, T, H, 512), dtype=torch.bfloat16, device=DEV)
    s["lse"] = torch.empty((B, T, H), dtype=torch.float32, device=DEV)
    s["miss"] = torch.empty((B,), dtype=torch.int32, device=DEV)
    if c["slots"]:
        for _ in range(RING):       # once round the ring: the slot pool reaches its steady state
            _run_step(s)
    return s


def _run_step(s):
    """the next decode step of one layer, and the write-back of its new entries where the program appends"""
    c, i, cache = s["case"], s["step"] % RING, s["cache"]
    s["step"] += 1
    s["ctx"].decode_step(cache, s["q"][i], s["w"], s["keys"], s["len"], s["q_attn"][i % ATTN_SETS], s["step"], s["idx"], s["out"],
                         s["lse"], s["miss"], block_table=s["table"])
    r = {"idx": s["idx"], "out": s["out"], "lse": s["lse"], "miss": s["miss"]}
    if c["append"]:
        s["ctx"].append(cache, s["new_key"][i], s["new_rows"][i], s["keys"], s["len"], s["step"], s["placed"],
                        s["new_scale"][i] if c["paged"] else None, s["table"])
        r.update(placed=s["placed"], len=s["len"], keys=s["keys"])
    if c["slots"] or c["append"]:
        r.update(slot_pool=cache.slot_pool, slot_of=cache.slot_of, token_of=cache.token_of, stamp=cache.stamp)
    return r


def _normal_index_inputs(c, seed):
    """queries and keys as a network gives them: normal, quantised to e4m3, head weights of either sign"""
    g = _gen(seed, 6)
    q = _e4m3(torch.randn((c["B"], c["T"], c["Hi"], c["Di"]), generator=g, device=DEV) * 4)
    w = torch.randn((c["B"], c["T"], c["Hi"]), generator=g, device=DEV) / 16
    keys = torch.empty((c["B"], c["L"], c["Di"]), dtype=torch.uint8, device=DEV)
    for b in range(c["B"]):
        keys[b] = _e4m3(torch.randn((c["L"], c["Di"]), generator=g, device=DEV) * 4)
    return q, w, keys


def _prepare_score(c, seed):
    q, w, keys = _normal_index_inputs(c, seed)
    return dict(kind="score", case=c, ctx=bnd.Context(_config(c)), q=q, w=w, keys=keys,
                len=torch.full((c["B"],), c["L"], dtype=torch.int32, device=DEV),
                score=torch.zeros((c["B"], c["T"], c["L"]), dtype=torch.float32, device=DEV))


def _run_score(s):
    s["ctx"].index_score(s["q"], s["w"], s["keys"], s["len"], s["score"])
    return s["score"]


def _prepare_select(c, seed):
    q, w = _index_queries(c, seed)
    keys, table = _key_store(c, seed)
    return dict(kind="select", case=c, step=0, ctx=bnd.Context(_config(c)), q=q, w=w, keys=keys, table=table, len=_lengths(c, seed),
                idx=torch.empty((c["B"], c["T"], c["k"]), dtype=torch.int32, device=DEV))


def _run_select(s):
    i = s["step"] % RING
    s["step"] += 1
    s["ctx"].index_topk(s["q"][i], s["w"], s["keys"], s["len"], s["idx"], s["table"])
    return s["idx"]


def _gather_selections(c, seed):
    """ring of selections [RING,B,T,k]: the largest values of a field that turns slowly, ascending"""
    g = _gen(seed, 7)
    a, b = (torch.randn((c["B"], c["L"]), generator=g, device=DEV) for _ in range(2))
    sets = []
    for s in range(RING + c["T"] - 1):
        angle = 4 * math.pi * s / RING
        sets.append((a * math.cos(angle) + b * math.sin(angle)).topk(c["k"], dim=1).indices.sort(dim=1).values.to(torch.int32))
    return torch.stack([torch.stack(sets[s:s + c["T"]], dim=1) for s in range(RING)])


def _prepare_gather(c, seed):
    B, T, k = c["B"], c["T"], c["k"]
    cfg = _config(c, slots_per_seq=c["slots"])
    s = dict(kind="gather", case=c, step=0, ctx=bnd.Context(cfg), sel=_gather_selections(c, seed),
             cache=bnd.Cache.allocate(cfg, B, host_pool=_host_pool(c, seed)),
             len=torch.full((B,), c["L"], dtype=torch.int32, device=DEV),
             slot=torch.empty((B, T, k), dtype=torch.int32, device=DEV),
             rows=torch.empty((B, T, k, _stride(c)), dtype=torch.uint8, device=DEV),
             miss=torch.empty((B,), dtype=torch.int32, device=DEV))
    s["ctx"].cache_reset(s["cache"], B)
    for _ in range(RING):
        _run_gather(s)
    return s


def _run_gather(s):
    i, cache = s["step"] % RING, s["cache"]
    s["step"] += 1
    s["ctx"].gather_latent(cache, s["sel"][i], s["len"], s["step"], s["slot"], s["rows"], s["miss"])
    return {"rows": s["rows"], "slot": s["slot"], "miss": s["miss"], "slot_of": cache.slot_of, "token_of": cache.token_of,
            "stamp": cache.stamp}


def _slot_lists(c, seed):
    """[B,T,k] distinct slots, ascending; a ragged list ends in -1"""
    g = _gen(seed, 8)
    lists = torch.rand((c["B"], c["T"], c["S"]), generator=g, device=DEV).topk(c["k"], dim=2).indices.sort(dim=2).values.to(torch.int32)
    if c["ragged"]:
        n = torch.randint(c["k"] // 4, c["k"] + 1, (c["B"], c["T"], 1), generator=g, device=DEV)
        lists = torch.where(torch.arange(c["k"], device=DEV) < n, lists, torch.full_like(lists, -1))
    return lists.contiguous()


def _mla_pool(c, seed, b):
    return _entries(_gen(seed, 2048 + b), c["S"], c["fmt"])


def _prepare_mla(c, seed):
    pool = torch.empty((c["B"], c["S"], _stride(c)), dtype=torch.uint8, device=DEV)
    for b in range(c["B"]):
        pool[b] = _mla_pool(c, seed, b)
    return dict(kind="mla", case=c, ctx=bnd.Context(_config(c)), pool=pool, list=_slot_lists(c, seed), q=_attn_queries(c, seed, 1)[0],
                out=torch.empty((c["B"], c["T"], c["H"], 512), dtype=torch.bfloat16, device=DEV),
                lse=torch.empty((c["B"], c["T"], c["H"]), dtype=torch.float32, device=DEV))


def _run_mla(s):
    s["ctx"].sparse_mla_decode(s["q"], s["pool"], s["list"], s["out"], s["lse"])
    return {"out": s["out"], "lse": s["lse"]}


# ------------------------------------------------------------------ the work of a pass, and what its results may differ by

def work(case):
    c = case
    B, T, kind = c["B"], c["T"], c["kind"]
    by = fl = 0.0
    if kind in ("step", "score", "select"):
        length = 0.5 * (c.get("lo", c["L"]) + c.get("hi", c["L"]))
        by += B * length * (c["Di"] + (4 if c.get("paged") else 0)) + B * T * c["Hi"] * (c["Di"] + 4)
        fl += 2.0 * B * T * length * c["Hi"] * (c["Di"] + 1)
        by += B * T * (4.0 * length if kind == "score" else 4.0 * c["k"])
    if kind in ("step", "mla"):
        k = min(c["k"], 0.5 * (c["lo"] + c["hi"])) if kind == "step" else c["k"] * (0.625 if c["ragged"] else 1.0)
        by += B * T * (k * _stride(c) + c["H"] * (1152 + 1024 + 4)) + (0 if kind == "step" else B * T * c["k"] * 4)
        fl += 2.0 * B * T * k * c["H"] * (576 + 512)
    if kind == "gather":
        by += B * T * c["k"] * (2.0 * _stride(c) + 8)
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] in ("select", "gather"):
        return "exact"
    if case["kind"] == "score":
        return {"rel": 7e-5}          # fp8 matrix instructions align their 128 products before adding them
    return {"rel": 1e-2, "max": 0.1}  # bf16 operands and results, fp32 sums


# ------------------------------------------------------------------ the same in 64 bits

def _scores(q, w, keys):
    """[T,L] from e4m3 bytes q [T,Hi,Di], keys [L,Di]"""
    kt = _value(keys).t().contiguous()
    return torch.stack([(w[t].to(torch.float64).unsqueeze(1) * torch.relu(_value(q[t]) @ kt)).sum(0) for t in range(q.shape[0])])


def _largest(score, vis, k):
    """the k largest of score[:vis], earlier positions first among equals, ascending, -1 padded"""
    n = min(vis, k)
    got = torch.full((k,), -1, dtype=torch.int64, device=DEV)
    got[:n] = score[:vis].sort(descending=True, stable=True).indices[:n].sort().values
    return got


def _attend(q, rows):
    """out [H,512], lse [H] of queries [H,576] over entries [n,576]"""
    z = (q.to(torch.float64) @ rows.t().contiguous()) * SCALE
    lse = torch.logsumexp(z, dim=1)
    return torch.exp(z - lse.unsqueeze(1)) @ rows[:, :512].contiguous(), lse


def exact(case, seed):
    return globals()["_exact_" + case["kind"]](case, seed)


def _exact_score(c, seed):
    q, w, keys = _normal_index_inputs(c, seed)
    return torch.stack([_scores(q[b], w[b], keys[b]) for b in range(c["B"])])


def _select_one(c, q, w, keys, scale, length):
    score = _scores(q, w, keys)
    if scale is not None:             # one float32 product of the exact sum, as the paged cache defines it
        score = (score.to(torch.float32) * scale).to(torch.float64)
    return torch.stack([_largest(score[t], max(length - (c["T"] - 1 - t), 0), c["k"]) for t in range(c["T"])])


def _exact_select(c, seed):
    q, w = _index_queries(c, seed)
    lens = _lengths(c, seed).tolist()
    scale = _pages(c, seed)[1] if c["paged"] else None
    return torch.stack([_select_one(c, q[0][b], w[b], _keys(c, seed, b), None if scale is None else scale[b], lens[b])
                        for b in range(c["B"])])


def _exact_gather(c, seed):
    sel = _gather_selections(c, seed)[0].long()
    return {"rows": torch.stack([_latents(c, seed, b)[sel[b]] for b in range(c["B"])]).to(torch.int64) if c["B"] * c["T"] <= 64 else None}


def _exact_mla(c, seed):
    lists, q = _slot_lists(c, seed), _attn_queries(c, seed, 1)[0]
    outs, lses = [], []
    for b in range(c["B"]):
        pool = _mla_pool(c, seed, b)
        for t in range(c["T"]):
            at = lists[b, t][lists[b, t] >= 0].long()
            o, l = _attend(q[b, t], _entry_values(pool[at], c["fmt"]))
            outs.append(o)
            lses.append(l)
    shape = (c["B"], c["T"], c["H"])
    return {"out": torch.stack(outs).view(*shape, 512), "lse": torch.stack(lses).view(shape)}


def _exact_step(c, seed):
    """the first pass after prepare(): step 0 of the ring, with RING steps behind it where the state was warmed up"""
    q, w = _index_queries(c, seed)
    q_attn = _attn_queries(c, seed, ATTN_SETS)
    lens = _lengths(c, seed)
    scale = _pages(c, seed)[1] if c["paged"] else None
    behind = RING if c["slots"] else 0
    new = _new_entries(c, seed) if c["append"] else None
    idx, outs, lses = [], [], []
    for b in range(c["B"]):
        keys, rows, length = _keys(c, seed, b), _latents(c, seed, b), int(lens[b])
        if new is not None and behind:
            n = min(behind * c["T"], c["L"] - length)
            at = slice(length, length + n)
            keys[at] = new[0][:, b].reshape(-1, c["Di"])[:n]
            rows[at] = new[2][:, b].reshape(-1, _stride(c))[:n]
            if scale is not None:
                scale[b, at] = new[1][:, b].reshape(-1)[:n]
            length += n
        got = _select_one(c, q[0][b], w[b], keys, None if scale is None else scale[b], length)
        idx.append(got)
        for t in range(c["T"]):
            o, l = _attend(q_attn[0, b, t], _entry_values(rows[got[t][got[t] >= 0]], c["fmt"]))
            outs.append(o)
            lses.append(l)
    shape = (c["B"], c["T"], c["H"])
    return {"idx": torch.stack(idx), "out": torch.stack(outs).view(*shape, 512), "lse": torch.stack(lses).view(shape)}
