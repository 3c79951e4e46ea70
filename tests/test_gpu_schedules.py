"""Which schedule an offloaded step takes under the switch, and that a fetch which travels with Attn0 in one launch changes
nothing but the time."""
import numpy as np
import pytest
import torch

from paper_2512_10576_amd import synth

pytestmark = pytest.mark.gpu


def _host(fmt, B, L):
    host = (synth.latent_rows_bf16, synth.latent_rows_fp8)[fmt](5, B * L)
    hp = torch.empty((B, L, host.shape[-1]), dtype=torch.uint8, pin_memory=True)
    hp.copy_(host.reshape(B, L, -1))
    return hp


def _moving_sets(B, T, L, k, moves):
    """selections that walk along a permutation of the positions: each misses as many entries as it moved"""
    perm = np.random.default_rng(7).permutation(L)
    at, out = 0, []
    for m in moves:
        at += m
        row = [np.sort(perm[(at + t * (m // 2) + np.arange(k)) % L]) for t in range(T)]
        out.append(torch.from_numpy(np.broadcast_to(np.stack(row), (B, T, k)).astype(np.int32).copy()).cuda())
    return out


class _Run:
    """decode steps of one context over the same inputs"""

    def __init__(self, fmt, B, T, H, k, L, S, flags, hp):
        from paper_2512_10576_amd import binding as b
        self.args = (B, T, H, k)
        self.ctx = b.Context(b.make_config(B, T, L, 4, 32, k, H, latent_fmt=fmt, slots_per_seq=S, flags=flags))
        self.cache = b.Cache.allocate(self.ctx.cfg, B, host_pool=hp)
        self.ctx.cache_reset(self.cache, B)
        qi, w, key = synth.indexer_inputs(5, B, T, 4, 32, L, 4, 4, 8)
        self.dev = [x.cuda() for x in (qi, w, key)] + [torch.full((B,), L, dtype=torch.int32, device="cuda")]
        self.miss = torch.empty((B,), dtype=torch.int32, device="cuda")
        self.step = 0

    def __call__(self, sel):
        B, T, H, k = self.args
        self.step += 1
        q = synth.attn_query(60 + self.step, B, T, H).cuda()
        idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
        out = torch.full((B, T, H, 512), 9.0, dtype=torch.bfloat16, device="cuda")
        lse = torch.full((B, T, H), 9.0, dtype=torch.float32, device="cuda")
        self.ctx.decode_step(self.cache, *self.dev, q, self.step, idx, out, lse, self.miss, sel)
        torch.cuda.synchronize()
        return [x.clone() for x in (out, lse, self.miss, self.cache.slot_of, self.cache.token_of, self.cache.stamp, self.cache.slot_pool)]


# fewer rows than twelve; twelve and more (Attn1 finishes the rows); lists too long for that; one row; several head groups of 32
@pytest.mark.parametrize("fmt,B,T,H,k", [(0, 3, 2, 128, 512), (1, 3, 1, 96, 300), (0, 16, 1, 128, 256), (1, 7, 2, 40, 256),
                                         (0, 2, 1, 128, 2100), (1, 14, 1, 16, 2100), (0, 1, 1, 128, 512)])
def test_fetch_that_travels_with_attn0(ess_lib, fmt, B, T, H, k):
    """Under the switch, once the miss counts are known, a short fetch and one long enough to be confined are carried by
    Attn0's launch (a short one is not counted as confined); outputs and cache state are those of the plain schedule, bit for bit."""
    from paper_2512_10576_amd import binding as b
    print("carried fetch", fmt, B, T, H, k, flush=True)
    L, S = 4 * T * k + 1000, 2 * T * k
    # everything misses; two steps that follow many misses; steps that follow few (the last one misses nothing)
    moves = [0, 2 * T * k, 2 * T * k, 4, 4, 0, 0]
    sets, hp = _moving_sets(B, T, L, k, moves), _host(fmt, B, L)
    auto, plain = _Run(fmt, B, T, H, k, L, S, b.ESS_FLAG_AUTO, hp), _Run(fmt, B, T, H, k, L, S, 0, hp)
    auto.ctx.set_overlap_threshold(1 << 20)                       # never split
    seen = []
    for sel in sets:
        x, y = auto(sel), plain(sel)
        seen.append((auto.ctx.last_overlap(), auto.ctx.last_carried(), auto.ctx.last_confined()))
        assert (plain.ctx.last_carried(), plain.ctx.last_confined()) == (False, 0)
        assert all(torch.equal(a, c) for a, c in zip(x, y)), seen
    assert int(auto.miss.sum()) == 0
    auto.ctx.close()
    plain.ctx.close()
    assert seen[0] == (0, False, 0), seen                         # no miss counts yet
    assert all(s == (0, True, 1) for s in seen[1:4]), seen        # the steps before missed everything: a long fetch is expected
    assert all(s == (0, True, 0) for s in seen[4:]), seen         # ... or next to nothing


def test_selfcheck_of_a_step_in_the_da_schedule(ess_lib):
    """The self-check hook on a step that would carry its fetch: the step takes tickets instead, and the check that is to fail
    fails, also where an earlier ticket-fed step of any size left its counters behind."""
    from paper_2512_10576_amd import binding as b
    B, T, H, k, L, S = 1, 1, 128, 512, 6000, 1100
    sets, hp = _moving_sets(B, T, L, k, [0, k, k, k, k]), _host(0, B, L)
    run = _Run(0, B, T, H, k, L, S, b.ESS_FLAG_AUTO, hp)
    run(sets[0])
    run.ctx.debug_ticket_grid(2048)               # thousands of tickets are drawn from Attn0's counters
    run(sets[1])
    assert (run.ctx.last_carried(), run.ctx.last_confined()) == (False, 1)
    run.ctx.debug_ticket_grid(0)
    run.ctx.selfcheck_inject(5000)
    run(sets[2])
    assert (run.ctx.last_carried(), run.ctx.last_confined()) == (False, 1)
    with pytest.raises(b.EssError) as err:
        run.ctx.get_stats()
    assert err.value.code == b.ESS_ERR_INTERNAL
    run(sets[3])
    assert run.ctx.get_stats()["steps"] == 4 and run.ctx.last_confined() == 0
    run.ctx.close()


@pytest.mark.parametrize("mask", [0x3F, 0x08, 0x20])
def test_timed_steps_take_the_schedule_of_untimed_ones(ess_lib, mask):
    """Timing the stages of a step whose fetch travels with Attn0 does not take it apart: the launch that holds both is
    booked as Attn0 (stage 3) and as the fetch (stage 5)."""
    from paper_2512_10576_amd import binding as b
    B, T, H, k, L, S = 4, 1, 128, 512, 6000, 1100
    sets, hp = _moving_sets(B, T, L, k, [0, k, k, 2]), _host(0, B, L)
    run = _Run(0, B, T, H, k, L, S, b.ESS_FLAG_AUTO, hp)
    run.ctx.set_overlap_threshold(1 << 20)
    run(sets[0])
    run.ctx.profile_enable(3, stage_mask=mask)
    for sel in sets[1:]:
        run(sel)
        assert run.ctx.last_carried()
    for ms in run.ctx.profile_read():
        assert (ms[3] > 0) == bool(mask & 0x08) and (ms[5] > 0) == bool(mask & 0x20)
        if mask == 0x3F:
            assert ms[5] <= ms[3]                                 # the marks are outside the pair
    run.ctx.close()


@pytest.mark.parametrize("fmt,B,T,k,with_attn0", [(0, 96, 1, 128, True), (0, 97, 1, 128, False), (1, 64, 4, 64, False), (1, 128, 1, 320, True),
                                                  (0, 100, 1, 2100, False)])
def test_short_fetch_goes_in_front_where_it_would_cost_attn0_a_round(ess_lib, fmt, B, T, k, with_attn0):
    """A carried fetch takes two of eight XCDs: where Attn0 has 193 to 256 workgroups (96 x 2 ranges; 97 x 2; 256 rows; 128; 100 x
    2 ranges) the 192 CUs left would do it in two rounds instead of one, and a short fetch runs in front of it.  Outputs and
    cache state are those of the plain schedule, bit for bit, either way."""
    from paper_2512_10576_amd import binding as b
    print("short fetch", fmt, B, T, k, flush=True)
    H, L, S = 128, 4 * T * k + 100, 2 * T * k
    sets, hp = _moving_sets(B, T, L, k, [0, 2, 2, 0]), _host(fmt, B, L)
    auto, plain = _Run(fmt, B, T, H, k, L, S, b.ESS_FLAG_AUTO, hp), _Run(fmt, B, T, H, k, L, S, 0, hp)
    auto.ctx.set_overlap_threshold(1 << 20)
    for i, sel in enumerate(sets):
        x, y = auto(sel), plain(sel)
        assert all(torch.equal(a, c) for a, c in zip(x, y)), i
        if i > 1:                                                 # (follow a step of few misses)
            assert (auto.ctx.last_carried(), auto.ctx.last_confined()) == (with_attn0, 0), i
    auto.ctx.close()
    plain.ctx.close()
