"""A resident decode step captured in a HIP graph: every replay is checked against the CPU oracle, with
new inputs copied into the captured buffers and ordinary eager work between the replays.  (An offloaded
step carries the step number, the LRU time stamp, as a launch argument, so a captured one would
repeat its stamp: callers update that argument or launch those steps eagerly.)"""
import numpy as np
import pytest
import torch

from oracle import ess_oracle as O
from paper_2512_10576_amd import synth
from tests.test_gpu_stages import _check_attn, _ctx, _qbits, _topk_sets_equal

pytestmark = pytest.mark.gpu


def test_resident_decode_step_replayed_from_a_graph(ess_lib):
    from paper_2512_10576_amd import binding as bnd
    print("graph capture of a resident decode step", flush=True)
    B, T, Hi, Di, L, k, H = 2, 2, 64, 128, 5000, 512, 128
    ctx_len = torch.tensor([5000, 3777], dtype=torch.int32)
    pool = synth.latent_rows_bf16(3, B * L).reshape(B, L, 1152)
    ctx = _ctx(ess_lib, max_batch=B, max_q_tokens=T, max_ctx=L, idx_heads=Hi, idx_dim=Di, topk=k, attn_heads=H)
    cache = bnd.Cache.allocate(ctx.cfg, B, slot_pool=pool.cuda())
    ctx.cache_reset(cache, B)
    qi0, w0, key = synth.indexer_inputs(10, B, T, Hi, Di, L, 8, 8, 16)
    dqi, dw, dkey, dlen = qi0.cuda(), w0.cuda(), key.cuda(), ctx_len.cuda()
    dq = synth.attn_query(10, B, T, H).cuda()
    idx_out = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
    out = torch.empty((B, T, H, 512), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((B, T, H), dtype=torch.float32, device="cuda")
    mc = torch.full((B,), 7, dtype=torch.int32, device="cuda")

    def reference(qi, w, q):
        oc = O.SlotCache(B, L, L)
        oc.make_resident_identity()
        return O.decode_step(qi.numpy(), w.numpy(), key.numpy(), ctx_len.numpy(), k, oc, pool.numpy().copy(), None,
                             _qbits(q), O.FMT_BF16, 576 ** -0.5, 1)

    # eager run first (also the warm-up the capture needs)
    ctx.decode_step(cache, dqi, dw, dkey, dlen, dq, 1, idx_out, out, lse, mc)
    torch.cuda.synchronize()
    r = reference(qi0, w0, dq.cpu())
    _topk_sets_equal(idx_out.cpu().numpy(), r["idx"])
    _check_attn(out, lse, r["out"], r["lse"])

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.decode_step(cache, dqi, dw, dkey, dlen, dq, 1, idx_out, out, lse, mc)
    for rep in range(3):
        print("  replay", rep, flush=True)
        qi, w, _ = synth.indexer_inputs(20 + rep, B, T, Hi, Di, 64, 8, 8, 16)      # new queries, same keys
        q = synth.attn_query(20 + rep, B, T, H)
        dqi.copy_(qi); dw.copy_(w); dq.copy_(q)
        out.zero_(); idx_out.zero_(); mc.fill_(9)                                   # eager work between the replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        r = reference(qi, w, q)
        _topk_sets_equal(idx_out.cpu().numpy(), r["idx"])
        _check_attn(out, lse, r["out"], r["lse"])
        assert mc.cpu().tolist() == [0, 0]
    ctx.close()


def _offloaded(ess_lib, B, T, L, S, k, H, flags):
    """a context with a cache whose entries are in host memory, and what restores and compares its state"""
    from paper_2512_10576_amd import binding as bnd
    host = torch.empty((B, L, 1152), dtype=torch.uint8, pin_memory=True)
    host.copy_(synth.latent_rows_bf16(7, B * L).reshape(B, L, 1152))
    ctx = _ctx(ess_lib, max_batch=B, max_q_tokens=T, max_ctx=L, idx_heads=64, idx_dim=128, topk=k, attn_heads=H, slots_per_seq=S,
               flags=flags)
    cache = bnd.Cache.allocate(ctx.cfg, B, host_pool=host)
    ctx.cache_reset(cache, B)
    return ctx, cache, [cache.slot_of, cache.token_of, cache.stamp, cache.slot_pool]


def _replays_match_eager(step, state, outputs, inputs, variants):
    """`step()` is captured once; then, for every variant of the inputs, an eager run and a replay from the same state:
    same outputs and same state afterwards, bit for bit, with the eager work between the replays"""
    before = [x.clone() for x in state]

    def once(run, values):
        for x, v in zip(state, before):
            x.copy_(v)
        for x, v in zip(inputs, values):
            x.copy_(v)
        for x in outputs:
            x.fill_(9)
        torch.cuda.synchronize()
        run()
        torch.cuda.synchronize()
        return [x.clone() for x in outputs + state]

    once(step, variants[0])
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for i, values in enumerate(variants):
        print("  replay", i, flush=True)
        eager = once(step, values)
        for n, (x, y) in enumerate(zip(eager, once(g.replay, values))):
            assert torch.equal(x, y), (i, n)
        again = once(step, values)                           # eager calls use the same events as the capture did
        assert all(torch.equal(x, y) for x, y in zip(eager, again)), i


@pytest.mark.parametrize("flags", ["plain", "auto", "auto, many misses", "split batch", "serial"])
def test_offloaded_decode_step_replayed_from_a_graph(ess_lib, flags):
    """The fork to the side stream, the events that kernels complete (recorded as nodes under capture) and the joins:
    a replay gives what an eager call with the same step number gives on the same state."""
    from paper_2512_10576_amd import binding as bnd
    print("graph capture of an offloaded decode step:", flags, flush=True)
    B, T, L, S, k, H = 4, 2, 9000, 3000, 512, 128
    flag = {"plain": 0, "split batch": bnd.ESS_FLAG_DBA, "serial": bnd.ESS_FLAG_SERIAL}.get(flags, bnd.ESS_FLAG_AUTO)
    ctx, cache, state = _offloaded(ess_lib, B, T, L, S, k, H, flag)
    qi, w, key = (x.cuda() for x in synth.indexer_inputs(5, B, T, 64, 128, L, 8, 8, 16))
    lens = torch.full((B,), L, dtype=torch.int32)
    sets = synth.TopkTrace(3, lens, T, k, 0.5 if flags == "auto, many misses" else 0.97)
    trace = [sets.next().cuda() for _ in range(6)]
    lens = lens.cuda()
    sel, q = trace[0].clone(), synth.attn_query(1, B, T, H).cuda()
    idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
    out = torch.empty((B, T, H, 512), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((B, T, H), dtype=torch.float32, device="cuda")
    miss = torch.empty((B,), dtype=torch.int32, device="cuda")

    def step(n):
        ctx.decode_step(cache, qi, w, key, lens, q, n, idx, out, lse, miss, topk_override=sel)

    for n in (1, 2):
        sel.copy_(trace[n - 1])
        step(n)
    variants = [(trace[2 + i], synth.attn_query(60 + i, B, T, H).cuda()) for i in range(4)]
    _replays_match_eager(lambda: step(3), state, [idx, out, lse, miss], [sel, q], variants)
    ctx.close()


@pytest.mark.parametrize("B,k", [(2, 300), (8, 2047)])       # in line, and (32 MiB of rows and more) on two streams
def test_gather_replayed_from_a_graph(ess_lib, B, k):
    print("graph capture of a gather", B, k, flush=True)
    T, L = 2, 9000
    ctx, cache, state = _offloaded(ess_lib, B, T, L, 5000, k, 8, 0)
    g = torch.Generator().manual_seed(1)
    order = torch.stack([torch.randperm(L, generator=g) for _ in range(B)])
    picks = [torch.stack([order[:, 50 * s + 25 * t:50 * s + 25 * t + k] for t in range(T)], dim=1).to(torch.int32).contiguous().cuda()
             for s in range(6)]
    lens = torch.full((B,), L, dtype=torch.int32, device="cuda")
    sel = picks[0].clone()
    slot = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
    rows = torch.empty((B, T, k, 1152), dtype=torch.uint8, device="cuda")
    miss = torch.empty((B,), dtype=torch.int32, device="cuda")
    ctx.gather_latent(cache, sel, lens, 1, slot, rows, miss)
    _replays_match_eager(lambda: ctx.gather_latent(cache, sel, lens, 2, slot, rows, miss), state, [slot, rows, miss], [sel],
                         [(p,) for p in picks[1:5]])
    assert 0 < int(miss.min()) and int(miss.max()) < k
    ctx.close()
