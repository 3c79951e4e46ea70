"""Look-up and LRU update where the kernel's work changes shape: pools that end inside a group of 64 slots or fill the last
one, more slots at the victims' threshold stamp than fit one list (a new pool), more misses than one list holds, stamps
older than 254 steps, selections that are not whole rounds of the workgroup, several bitmap words a thread.  And the selected
rows, whose gather shares a launch with the fetch from 32 MiB of them on (odd batch, ragged last workgroups)."""
import numpy as np
import pytest
import torch

from oracle import ess_oracle as O
from paper_2512_10576_amd import synth

pytestmark = pytest.mark.gpu

CASES = [  # max_ctx, slots, k, T, kept share of the selection, first step
    (300, 40, 16, 2, 0.5, 1),             # one group of slots, not full
    (4000, 1025, 1024, 1, 0.3, 1),        # one slot in the second group of a wave's range
    (32768, 3072, 2048, 1, 0.9, 1),       # whole groups; full after six steps
    (32768, 3072, 2048, 1, 0.9, 300),     # first used when a stamp of 0 has no digit of its own
    (32768, 6144, 2048, 1, 0.55, 1),      # more slots at the threshold than a list holds, fewer misses than that
    (40000, 5000, 2048, 2, 0.8, 250),     # the digits end among these steps
    (40000, 16384, 2048, 2, 0.1, 1),      # the largest pool with its stamps in registers, more than 1024 misses
    (131072, 6553, 2048, 2, 0.9, 70000),  # four bitmap words a thread, odd pool
    (70001, 4001, 1000, 3, 0.85, 7),      # three bitmap words: rounded to four; lists read the table again
]


@pytest.mark.parametrize("L,S,k,T,kept,first", CASES)
def test_lookup_and_update_against_oracle(ess_lib, L, S, k, T, kept, first):
    from paper_2512_10576_amd import binding as bnd
    print("bookkeeping:", L, S, k, T, kept, first, flush=True)
    B = 2
    hp = torch.empty((B, L, 656), dtype=torch.uint8, pin_memory=True)
    hp.copy_(torch.randint(0, 256, (L, 656), generator=torch.Generator().manual_seed(4), dtype=torch.uint8))
    hp[1].add_(1)                           # sequences differ
    ctx_len = torch.tensor([L, L - 7], dtype=torch.int32)
    ctx = bnd.Context(bnd.make_config(max_batch=B, max_q_tokens=T, max_ctx=L, idx_heads=4, idx_dim=32, topk=k, attn_heads=8,
                                      slots_per_seq=S, latent_fmt=1))
    cache = bnd.Cache.allocate(ctx.cfg, B, host_pool=hp)
    ctx.cache_reset(cache, B)
    oc = O.SlotCache(B, L, S)
    trace = synth.TopkTrace(9, ctx_len, T, k, kept, zipf_s=0.2)
    slot_idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
    rows = torch.empty((B, T, k, 656), dtype=torch.uint8, device="cuda")
    mc = torch.empty((B,), dtype=torch.int32, device="cuda")
    for step in range(first, first + 14):
        idx = trace.next()
        if step == first + 5:
            idx[1] = -1                   # a sequence that selects nothing
        r = oc.step(idx.numpy(), step)
        ctx.gather_latent(cache, idx.cuda(), ctx_len.cuda(), step, slot_idx, rows, mc)
        torch.cuda.synchronize()
        assert np.array_equal(mc.cpu().numpy(), r["miss_count"]), step
        assert np.array_equal(slot_idx.cpu().numpy(), r["slot_idx"]), step
        assert np.array_equal(cache.token_of.cpu().numpy(), oc.token_of), step
        assert np.array_equal(cache.stamp.cpu().numpy().astype(np.int64), oc.stamp.astype(np.int64)), step
        # the rows of the selection, gathered beside the fetch and behind it: bytes of the host pool, zeros where nothing is selected
        sel = idx.long()
        want = torch.stack([hp[b][sel[b].clamp(min=0)] for b in range(B)])
        want[sel < 0] = 0
        assert torch.equal(rows.cpu(), want), step
    ctx.close()


@pytest.mark.parametrize("B,k,missing", [(27, 2047, 2047), (13, 2600, 40), (13, 2600, 0)])
def test_rows_gathered_beside_the_fetch(ess_lib, B, k, missing):
    """every entry fetched, a few, none; rows that end inside a workgroup's share"""
    from paper_2512_10576_amd import binding as bnd
    print("rows beside the fetch:", B, k, missing, flush=True)
    L, S = 6000, 2700
    assert B * k * 1152 >= 32 << 20
    hp = torch.empty((B, L, 1152), dtype=torch.uint8, pin_memory=True)
    hp.copy_(torch.randint(0, 256, (B, L, 1152), generator=torch.Generator().manual_seed(4), dtype=torch.uint8))
    ctx = bnd.Context(bnd.make_config(max_batch=B, max_q_tokens=1, max_ctx=L, idx_heads=4, idx_dim=32, topk=k, attn_heads=8,
                                      slots_per_seq=S, latent_fmt=0))
    cache = bnd.Cache.allocate(ctx.cfg, B, host_pool=hp)
    ctx.cache_reset(cache, B)
    ctx_len = torch.full((B,), L, dtype=torch.int32, device="cuda")
    slot_idx = torch.empty((B, 1, k), dtype=torch.int32, device="cuda")
    rows = torch.empty((B, 1, k, 1152), dtype=torch.uint8, device="cuda")
    mc = torch.empty((B,), dtype=torch.int32, device="cuda")
    for step in range(1, 4):
        idx = (torch.arange(k, dtype=torch.int32) + (step - 1) * missing) % L
        idx = idx.expand(B, 1, k).contiguous()
        idx[B - 1, 0, k // 2] = -1
        rows.fill_(7)
        ctx.gather_latent(cache, idx.cuda(), ctx_len, step, slot_idx, rows, mc)
        torch.cuda.synchronize()
        assert int(mc[0]) == (k if step == 1 else missing), step
        want = hp[:, idx[0, 0].long()].clone()
        want[B - 1, k // 2] = 0
        assert torch.equal(rows.cpu()[:, 0], want), step
    ctx.close()
