"""GPU parity at the edges of the ranges that attention, top-k and the schedules divide their work by: list lengths
around whole tiles and splits, head counts around a wave's 32, rows around the candidate list's size, gathered rows
beside a fetch, and a fetch in line with attention against one beside it."""
import numpy as np
import pytest
import torch

from oracle import ess_oracle as O
from paper_2512_10576_amd import synth
from tests.test_gpu_stages import _check_attn, _ctx, _qbits, _run_topk, _topk_sets_equal

pytestmark = pytest.mark.gpu


# lengths: nothing, one entry, a tile of 32 less and more, tiles that do not divide by the split count
@pytest.mark.parametrize("fmt", [O.FMT_BF16, O.FMT_FP8])
@pytest.mark.parametrize("B,T,H,k,lens", [
    (1, 1, 128, 2048, [2048]),                            # many splits of one row, merged by four waves
    (1, 1, 5, 65, [65]),
    (3, 2, 40, 160, [0, 1, 31, 32, 33, 160]),             # a second wave with eight heads
    (2, 2, 33, 97, [96, 97, 64, 63]),
    (5, 1, 128, 300, [300, 0, 129, 128, 299]),
    (65, 4, 16, 96, [96, 95, 0, 32]),                     # 260 rows: one split, no empty workgroup left over
])
def test_attention_list_lengths_and_heads(ess_lib, fmt, B, T, H, k, lens):
    print("attention ranges", fmt, B, T, H, k, flush=True)
    S = max(512, k)
    rng = np.random.default_rng(B * 1000 + H)
    rows = synth.latent_rows_bf16(B, B * S) if fmt == O.FMT_BF16 else synth.latent_rows_fp8(B, B * S)
    pool = rows.reshape(B, S, -1)
    q = synth.attn_query(H, B, T, H)
    idx = np.full((B, T, k), -1, np.int32)
    for i in range(B * T):
        n = lens[i % len(lens)]
        idx[i // T, i % T, :n] = rng.choice(S, n, replace=False)
    if k > 2:
        idx[0, 0, 1] = -1                                 # a hole
    scale = 1 / 24
    some = sorted({0, 1, 2, B - 2, B - 1} & set(range(B)))     # the oracle on the first sequences and the last
    ref_out, ref_lse = O.sparse_mla(_qbits(q[some]), pool[some].numpy(), idx[some], fmt, scale)
    ctx = _ctx(ess_lib, max_batch=B, max_q_tokens=T, max_ctx=S, idx_heads=4, idx_dim=32, topk=k, attn_heads=H, latent_fmt=fmt,
               sm_scale=scale)
    out = torch.full((B, T, H, 512), 9.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, T, H), 9.0, dtype=torch.float32, device="cuda")
    ctx.sparse_mla_decode(q.cuda(), pool.cuda(), torch.from_numpy(idx).cuda(), out, lse)
    torch.cuda.synchronize()
    ctx.close()
    # lists of a handful of quantised entries: few bf16-rounded weights, which do not average out (2^-8 of the values)
    err = np.abs(out[some].float().cpu().numpy() - ref_out)
    assert np.all(err <= 2e-2 + 2e-2 * np.abs(ref_out)), err.max()
    short = (idx[some] >= 0).sum(-1) < 64
    if not short.all():
        long_rows = ~short
        _check_attn(out[some][torch.from_numpy(long_rows)], lse[some][torch.from_numpy(long_rows)], ref_out[long_rows], ref_lse[long_rows])
    # the log-sum-exp of every row: no rounded weights in it.  Of one entry it is the logit itself: with quantised entries,
    # whose dequantised values are rounded to bf16 (2^-9 of each at most, 2^-9 / sqrt(3) in the mean square), the sum over
    # 512 products of N(0,1) values is off by scale * 2^-9 / sqrt(3) * sqrt(512) = 1.1e-3 in the mean square; six times that
    atol = 2e-3 if fmt == O.FMT_BF16 else 6 * scale * 2.0 ** -9 * (512 / 3) ** 0.5
    got_lse, fin = lse[some].cpu().numpy().astype(np.float64), np.isfinite(ref_lse)
    assert np.array_equal(np.isneginf(got_lse), np.isneginf(ref_lse))
    assert np.allclose(got_lse[fin], ref_lse[fin], atol=atol, rtol=1e-4), np.abs(got_lse[fin] - ref_lse[fin]).max()


@pytest.mark.parametrize("k", [64, 2048])
def test_attention_of_an_infinite_value_with_weight_zero(ess_lib, k):
    """An entry that is infinite in one column, where every query is negative: its logit is -inf, its weight zero, and
    zero times infinity is no number -- in that column alone.  The others, values beyond the fp16 range among them, are
    what they are without it (the plain average of identical entries, exact)."""
    print("attention, infinite value", k, flush=True)
    B, T, H, L = 1, 2, 128, 2048
    rows = torch.zeros((B, L, 576), dtype=torch.bfloat16)
    rows[..., 0], rows[..., 1] = 3.0e5, -0.5
    rows[0, 3, 7] = float("inf")
    q = torch.zeros((B, T, H, 576), dtype=torch.bfloat16)
    q[..., 7] = -1.0
    idx = torch.arange(k, dtype=torch.int32).expand(B, T, k).contiguous()
    ctx = _ctx(ess_lib, max_batch=B, max_q_tokens=T, max_ctx=L, idx_heads=4, idx_dim=32, topk=k, attn_heads=H)
    out = torch.full((B, T, H, 512), 9.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, T, H), 9.0, dtype=torch.float32, device="cuda")
    ctx.sparse_mla_decode(q.cuda(), rows.view(torch.uint8).reshape(B, L, 1152).cuda(), idx.cuda(), out, lse)
    torch.cuda.synchronize()
    ctx.close()
    want = torch.zeros((B, T, H, 512))
    want[..., 0], want[..., 1], want[..., 7] = rows[0, 0, 0].float(), -0.5, float("nan")
    assert torch.equal(out.float().cpu().nan_to_num(nan=-12345.0), want.nan_to_num(nan=-12345.0)), out[0, 0, 0, :9]
    assert np.allclose(lse.cpu().numpy(), np.log(k - 1), atol=1e-4)


# rows around k, a thread's eight keys, the candidate list (8192) and the sampled path above it
@pytest.mark.parametrize("kind", ["distinct", "ties", "one value", "low and high", "power of two"])
@pytest.mark.parametrize("vis,k", [(9, 8), (1025, 1024), (4097, 2048), (4096, 2048), (8191, 2048), (8192, 4096), (8193, 2048), (16384, 513)])
def test_topk_short_rows(ess_lib, kind, vis, k):
    print("topk", kind, vis, k, flush=True)
    rng = np.random.default_rng(vis)
    sc = rng.standard_normal((1, 1, vis)).astype(np.float32) * 100
    if kind == "ties":
        sc = np.round(sc / 64).astype(np.float32)         # a dozen values: thousands of equal scores
    elif kind == "one value":
        sc[:] = np.float32(-3.5)
    elif kind == "low and high":                          # the k-th largest among the lowest value, infinities and NaN
        sc[:] = np.float32(-np.inf)
        sc[0, 0, rng.choice(vis, k - 3, replace=False)] = rng.standard_normal(k - 3).astype(np.float32)
        sc[0, 0, 1] = np.float32(np.inf)
        sc[0, 0, 2] = np.float32(np.nan)
    elif kind == "power of two":                          # the k-th largest is the lower end of a histogram bin
        order = np.argsort(-sc[0, 0], kind="stable")
        sc[0, 0, order] = np.round(np.linspace(512 + k / 8, 512 - (vis - k) / 8, vis)).astype(np.float32)
        assert np.sort(sc[0, 0])[-k] == 512
    lens = np.array([vis])
    _topk_sets_equal(_run_topk(ess_lib, sc, [vis], k, 1), O.topk(sc, lens, k))


def test_topk_short_rows_of_a_long_context(ess_lib):
    """Contexts from 65536 share their rows: those that fit the candidate list are done by the candidate pass, the
    shortest, and those with too many ties, by the finishing kernel; and nothing of a call is left for the next."""
    print("topk, short rows of a long context", flush=True)
    rng = np.random.default_rng(3)
    L, k = 65536, 2048
    lens = [4096, 65536, 4097, 8192, 8193, 2048, 100, 0, 8000, 6000, 30000, 5000]
    B = len(lens)
    ctx = _ctx(ess_lib, max_batch=B, max_q_tokens=1, max_ctx=L, idx_heads=4, idx_dim=32, topk=k, attn_heads=8)
    for turn in range(4):
        sc = (rng.standard_normal((B, 1, L)) * 100).astype(np.float32)
        if turn % 2:
            sc = np.round(sc)
        sc[8] = np.round(sc[8] / 64)                         # a dozen values: thousands of equal scores
        idx = torch.full((B, 1, k), -5, dtype=torch.int32, device="cuda")
        ctx.topk(torch.from_numpy(sc).cuda(), torch.tensor(lens, dtype=torch.int32).cuda(), idx)
        torch.cuda.synchronize()
        _topk_sets_equal(idx.cpu().numpy(), O.topk(sc, np.array(lens), k))
        lens = lens[1:] + lens[:1]                           # another length for every row of the next call
    ctx.close()


@pytest.mark.parametrize("L", [9000, 65536])                 # one kernel, two kernels
def test_topk_of_short_rows_by_ticket(ess_lib, L):
    """Short rows of a longer context in the split-batch schedule with confined fetches, where the top-k of the second
    half takes its rows by ticket: the selections of the plain schedule."""
    from paper_2512_10576_amd import binding as bnd
    print("topk by ticket", L, flush=True)
    B, T, k, H, S = 8, 1, 512, 16, 2048
    host = torch.zeros((B, L, 656), dtype=torch.uint8, pin_memory=True)
    lens = torch.tensor([4097, L, 8192, 4096, 8192, 5000, L, 600], dtype=torch.int32).cuda()
    key = synth.indexer_inputs(1, B, T, 64, 128, L, 8, 8, 16)[2].cuda()
    qws = [tuple(x.cuda() for x in synth.indexer_inputs(30 + s, B, T, 64, 128, 64, 8, 8, 16)[:2]) for s in range(3)]
    q = synth.attn_query(9, B, T, H).cuda()
    results, confined = {}, []
    for flags in (0, bnd.ESS_FLAG_AUTO):
        ctx = _ctx(ess_lib, max_batch=B, max_q_tokens=T, max_ctx=L, idx_heads=64, idx_dim=128, topk=k, attn_heads=H,
                   latent_fmt=O.FMT_FP8, slots_per_seq=S, flags=flags)
        if flags:
            ctx.set_overlap_threshold(0)
        cache = bnd.Cache.allocate(ctx.cfg, B, host_pool=host)
        ctx.cache_reset(cache, B)
        got = []
        for step in range(3):
            idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
            out = torch.empty((B, T, H, 512), dtype=torch.bfloat16, device="cuda")
            ctx.decode_step(cache, *qws[step], key, lens, q, step + 1, idx, out)
            torch.cuda.synchronize()
            if flags:
                confined.append((ctx.last_overlap(), ctx.last_confined()))
            got.append(idx)
        results[flags] = got
        ctx.close()
    assert all(mode == 1 and n >= 1 for mode, n in confined[1:]), confined
    assert all(torch.equal(a, b) for a, b in zip(results[0], results[bnd.ESS_FLAG_AUTO]))


# (the last two: 32 MiB of rows and more, gathered on two streams beside the fetch; with quantised entries the rows of
# concurrent kernels share cache lines)
@pytest.mark.parametrize("fmt,B,T,L,S,k", [
    (O.FMT_BF16, 1, 1, 300, 40, 17), (O.FMT_BF16, 3, 2, 1000, 257, 100), (O.FMT_BF16, 2, 4, 3000, 1500, 333),
    (O.FMT_FP8, 1, 1, 300, 40, 17), (O.FMT_FP8, 3, 2, 1000, 257, 100),
    (O.FMT_BF16, 8, 2, 9000, 5000, 2047), (O.FMT_FP8, 13, 2, 9000, 5000, 2047)])
def test_gathered_rows_beside_a_fetch(ess_lib, fmt, B, T, L, S, k):
    """the rows of resident and of fetched entries, entry counts that are no multiple of a wave's sixteen"""
    from paper_2512_10576_amd import binding as bnd
    print("gather ranges", fmt, B, T, L, S, k, flush=True)
    rng = np.random.default_rng(L)
    src = (synth.latent_rows_bf16 if fmt == O.FMT_BF16 else synth.latent_rows_fp8)(L, B * L)
    stride = src.shape[-1]
    host = torch.empty((B, L, stride), dtype=torch.uint8, pin_memory=True)
    host.copy_(src.reshape(B, L, stride))
    ctx = _ctx(ess_lib, max_batch=B, max_q_tokens=T, max_ctx=L, idx_heads=4, idx_dim=32, topk=k, attn_heads=8, latent_fmt=fmt,
               slots_per_seq=max(S, T * k))
    cache = bnd.Cache.allocate(ctx.cfg, B, host_pool=host)
    ctx.cache_reset(cache, B)
    lens = torch.full((B,), L, dtype=torch.int32, device="cuda")
    slot = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
    rows = torch.empty((B, T, k, stride), dtype=torch.uint8, device="cuda")
    miss = torch.empty((B,), dtype=torch.int32, device="cuda")
    idx = None
    for step in range(1, 5):
        # after the first step about half of every list was selected by the step before: both gathers have rows to copy
        new = np.stack([np.stack([rng.permutation(L)[:k] for _ in range(T)]) for _ in range(B)]).astype(np.int32)
        if idx is not None:
            for b in range(B):
                for t in range(T):
                    old = idx[b, t][idx[b, t] >= 0][:k // 2]
                    fresh = new[b, t][~np.isin(new[b, t], old)]
                    new[b, t] = rng.permutation(np.concatenate([old, fresh])[:k])
        idx = new
        idx[:, :, step::7] = -1
        rows.fill_(0xEE)
        ctx.gather_latent(cache, torch.from_numpy(idx).cuda(), lens, step, slot, rows, miss)
        torch.cuda.synchronize()
        want = np.zeros((B, T, k, stride), np.uint8)
        for b in range(B):
            v = idx[b] >= 0
            want[b][v] = host[b].numpy()[idx[b][v]]
            if step > 1:
                assert 0 < int(miss[b]) < np.unique(idx[b][v]).size
        assert np.array_equal(rows.cpu().numpy(), want), step
    ctx.close()


@pytest.mark.parametrize("B,T,fmt", [(3, 2, O.FMT_FP8), (2, 1, O.FMT_BF16)])
def test_short_fetch_in_line_gives_the_bits_of_the_overlapped_schedule(ess_lib, B, T, fmt):
    """With few misses the switch keeps everything on the caller's stream, the fetch in Attn0's launch; the plain schedule runs
    Attn0 on the side stream: same outputs and cache state, bit for bit."""
    from paper_2512_10576_amd import binding as bnd
    print("short fetch", B, T, fmt, flush=True)
    L, k, H, S = 9000, 512, 128, 4 * 512 * T
    rows = synth.latent_rows_bf16 if fmt == O.FMT_BF16 else synth.latent_rows_fp8
    host = rows(5, B * L)
    hp = torch.empty((B, L, host.shape[-1]), dtype=torch.uint8, pin_memory=True)
    hp.copy_(host.reshape(B, L, -1))
    qi, w, key = (x.cuda() for x in synth.indexer_inputs(5, B, T, 64, 128, L, 8, 8, 16))
    lens = torch.full((B,), L, dtype=torch.int32)
    sets = synth.TopkTrace(3, lens, T, k, 0.97)
    trace = [sets.next().cuda() for _ in range(4)]
    lens = lens.cuda()
    results = {}
    for flags in (bnd.ESS_FLAG_AUTO, 0):
        ctx = _ctx(ess_lib, max_batch=B, max_q_tokens=T, max_ctx=L, idx_heads=64, idx_dim=128, topk=k, attn_heads=H, latent_fmt=fmt,
                   slots_per_seq=S, flags=flags)
        cache = bnd.Cache.allocate(ctx.cfg, B, host_pool=hp)
        ctx.cache_reset(cache, B)
        ctx.profile_enable(4)
        idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
        out = torch.empty((B, T, H, 512), dtype=torch.bfloat16, device="cuda")
        lse = torch.empty((B, T, H), dtype=torch.float32, device="cuda")
        miss = torch.empty((B,), dtype=torch.int32, device="cuda")
        got = []
        for step in range(4):
            q = synth.attn_query(50 + step, B, T, H).cuda()
            ctx.decode_step(cache, qi, w, key, lens, q, step + 1, idx, out, lse, miss, topk_override=trace[step])
            torch.cuda.synchronize()
            assert ctx.last_overlap() == 0
            # in line, Attn0 (stage 3) is timed on the caller's stream; beside the fetch's own launch it runs on the side stream.
            # The first step knows no miss counts yet: nothing tells that its fetch is short; the second follows a step
            # that fetched everything
            in_line = 3 in [stage for _, stage in ctx.profile_intervals(step)]
            if step != 1:
                assert in_line == (flags == bnd.ESS_FLAG_AUTO and step > 1), (flags, step)
            got.append([x.clone() for x in (out, lse, miss, cache.slot_of, cache.token_of, cache.stamp, cache.slot_pool)])
        assert int(miss.sum()) > 0
        ctx.close()
        results[flags] = got
    for a, b in zip(results[bnd.ESS_FLAG_AUTO], results[0]):
        for x, y in zip(a, b):
            assert torch.equal(x, y)


# Steps with gaps between them, few and many entries in turn: victims never used, of one stamp or of many, some or all of
# them older than the 254 steps that the one-pass threshold search tells apart, so that one or more passes over the older
# ones follow; more victims than a workgroup has threads; lists of whole rounds of the workgroup and others; a pool too
# large for the registers.  "late": a pool whose first step is past 255.
FROM_ONE = [1, 2, 3, 5, 90, 250, 254, 255, 256, 257, 258, 300, 301, 302, 303, 304, 560, 561, 562, 65530, 65535, 65536, 65537,
            65700, 65701, 65950, (1 << 24) + 3, (1 << 24) + 4]
LATE = [300, 301, 302, 303, 428, 429, 430, 509, 510, 511, 512, 556, 813, 814, 40000, 40001, 40127, 40128, 40129, 40400, (1 << 20) + 5,
        (1 << 20) + 6, (1 << 20) + 132, (1 << 20) + 133, (1 << 20) + 134, (1 << 32) - 300, (1 << 32) - 173, (1 << 32) - 1]


@pytest.mark.parametrize("steps", [FROM_ONE, LATE], ids=["from one", "late"])
@pytest.mark.parametrize("T,k,S,L", [(1, 100, 257, 1500), (1, 1024, 1500, 6000), (2, 1024, 4096, 9000), (2, 1000, 2500, 9000),
                                     (1, 1500, 17000, 30000)])
def test_bookkeeping_of_old_stamps(ess_lib, T, k, S, L, steps):
    from paper_2512_10576_amd import binding as bnd
    print("old stamps", T, k, S, L, steps[0], flush=True)
    B = 2
    host = torch.empty((B, L, 1152), dtype=torch.uint8, pin_memory=True)
    host.zero_()
    ctx = _ctx(ess_lib, max_batch=B, max_q_tokens=T, max_ctx=L, idx_heads=4, idx_dim=32, topk=k, attn_heads=8, slots_per_seq=S)
    cache = bnd.Cache.allocate(ctx.cfg, B, host_pool=host)
    ctx.cache_reset(cache, B)
    oc = O.SlotCache(B, L, S)
    rng = np.random.default_rng(S)
    lens = torch.full((B,), L, dtype=torch.int32, device="cuda")
    slot = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
    rows = torch.empty((B, T, k, 1152), dtype=torch.uint8, device="cuda")
    for i, step in enumerate(steps):
        n = k if i % 3 == 2 else max(1, k // 5)
        idx = np.full((B, T, k), -1, np.int32)
        for b in range(B):
            held = np.nonzero(oc.slot_of[b] >= 0)[0]
            for t in range(T):
                old = rng.choice(held, min(n // 3, held.size), replace=False) if held.size else held
                rest = rng.choice(np.setdiff1d(np.arange(L), old), n - old.size, replace=False)
                idx[b, t, :n] = rng.permutation(np.concatenate([old, rest]))
        r = oc.step(idx, step)
        ctx.gather_latent(cache, torch.from_numpy(idx).cuda(), lens, step, slot, rows)
        torch.cuda.synchronize()
        assert np.array_equal(slot.cpu().numpy(), r["slot_idx"]), step
        assert np.array_equal(cache.slot_of.cpu().numpy(), oc.slot_of), step
        assert np.array_equal(cache.token_of.cpu().numpy(), oc.token_of), step
        assert np.array_equal(cache.stamp.cpu().numpy().view(np.uint32), oc.stamp), step
    ctx.close()
