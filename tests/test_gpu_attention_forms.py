"""The attention kernel with 32 heads per workgroup (few rows, short lists, few heads; Attn1 that finishes its rows) at the
edges of its tiles, lists, head groups and ranges, against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import ess_oracle as O
from paper_2512_10576_amd import synth

pytestmark = pytest.mark.gpu


def _qbits(q):
    return q.view(torch.int16).cpu().numpy().view(np.uint16)


def _check(out, lse, ref_out, ref_lse, lse_tol=1e-4):
    """Weights are rounded to bf16 (2^-9 each, independent) and so is the output (2^-9): the error of a row's outputs is
    below 2^-8 of their size in the 2-norm, which 1e-2 bounds; logits and sums are fp32."""
    got, lg = out.float().cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isneginf(lg), np.isneginf(ref_lse))
    empty = np.isneginf(ref_lse)
    assert np.all(got[empty] == 0.0)
    assert np.linalg.norm(got - ref_out) <= 1e-2 * max(np.linalg.norm(ref_out), 1e-30)
    # row by row: a list of few entries has no averaging, its outputs are O(1) and off by 2^-8 of the largest
    assert np.all(np.abs(got - ref_out).max(-1) <= 2.0 ** -6 * np.maximum(np.abs(ref_out).max(-1), 1e-30))
    assert np.allclose(lg[~empty], ref_lse[~empty], atol=lse_tol, rtol=1e-5)


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("B,T,H,k,kind", [
    (1, 1, 128, 64, "full"), (2, 2, 16, 33, "ragged"), (1, 1, 40, 1, "full"), (64, 1, 128, 48, "ragged"), (1, 1, 1, 65, "full"), (1, 2, 31, 128, "full"), (2, 1, 33, 129, "ragged"), (1, 1, 128, 2048, "full"),
    (3, 1, 40, 513, "holes"), (1, 4, 16, 1000, "ragged"), (9, 1, 64, 191, "ragged"), (64, 1, 16, 320, "ragged"),
    (130, 1, 20, 192, "ragged"), (2, 2, 128, 514, "unaligned")])
def test_lists_heads_and_ranges(ess_lib, fmt, B, T, H, k, kind):
    """full; ragged: lists of every length from none up, -1 behind; holes: -1, and slots past the pool, between valid
    entries; unaligned: the list starts four bytes into an allocation."""
    from paper_2512_10576_amd import binding as b
    print("attention forms", fmt, B, T, H, k, kind, flush=True)
    S = max(k, 300) + 37
    stride = (1152, 656)[fmt]
    pool = (synth.latent_rows_bf16, synth.latent_rows_fp8)[fmt](7 * B + k, B * S).reshape(B, S, stride)
    rng = np.random.default_rng(B * 1000 + k)
    idx = np.stack([rng.permutation(S)[:k] for _ in range(B * T)]).astype(np.int32).reshape(B, T, k)
    ref = idx.copy()
    if kind == "ragged":
        for r, row in enumerate(idx.reshape(B * T, k)):
            n = (0, 1, 63, 64, 65, k - 1, k)[r] if r < 7 else int(rng.integers(0, k + 1))
            row[n:] = -1
        ref = idx.copy()
    if kind == "holes":
        hole = rng.random(idx.shape) < 0.3
        hole[..., 64:128] = True                                  # a tile without an entry
        ref[hole] = -1
        idx[hole] = np.where(rng.random(int(hole.sum())) < 0.5, -1, S + 5)
    q = synth.attn_query(3 + k, B, T, H)
    ctx = b.Context(b.make_config(B, T, S, 4, 32, k, H, latent_fmt=fmt, slots_per_seq=S))
    dev = torch.empty((B * T * k + 1,), dtype=torch.int32, device="cuda")
    at = 1 if kind == "unaligned" else 0
    lists = dev[at:at + B * T * k].view(B, T, k)
    lists.copy_(torch.from_numpy(idx))
    out = torch.full((B, T, H, 512), 9.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, T, H), 9.0, dtype=torch.float32, device="cuda")
    ctx.sparse_mla_decode(q.cuda(), pool.cuda(), lists, out, lse)
    torch.cuda.synchronize()
    ro, rl = O.sparse_mla(_qbits(q), pool.numpy(), ref, fmt, 576 ** -0.5)
    _check(out, lse, ro, rl)
    ctx.close()


@pytest.mark.parametrize("fmt,scale", [(0, 0.5), (1, 0.5), (0, 8.0)])
def test_reference_moves_from_tile_to_tile(ess_lib, fmt, scale):
    """Lists in the order of one head's logits, which grow by far more than 2^8 from tile to tile (a peaky softmax): the
    accumulators are rescaled in half the tiles of that head or more, and the other heads of the row move at other tiles.  128 rows of two
    workgroups: one range a row, all its tiles behind one another."""
    from paper_2512_10576_amd import binding as b
    B, T, H, k = 32, 4, 48, 640
    stride = (1152, 656)[fmt]
    pool = (synth.latent_rows_bf16, synth.latent_rows_fp8)[fmt](5, B * k).reshape(B, k, stride)
    q = synth.attn_query(8, B, T, H)
    z = np.matmul(O.decode_bf16(_qbits(q)), O.decode_rows(pool.numpy(), fmt).transpose(0, 2, 1)[:, None]) * (scale * np.log2(np.e))
    idx = np.empty((B, T, k), np.int32)
    for r in range(B * T):
        row = z.reshape(B * T, H, k)[r]
        order = np.argsort(row[r % H])
        idx.reshape(B * T, k)[r] = order
        tiles = row[:, order].reshape(H, k // 64, 64).max(-1)
        ref, moved = tiles[:, 0].copy(), np.zeros((H, k // 64), bool)
        for t in range(1, k // 64):                               # what the kernel does with the reference, 8 = kLazyMax
            moved[:, t] = tiles[:, t] > ref + 8
            ref = np.where(moved[:, t], tiles[:, t], ref)
        assert moved[r % H].sum() >= 4 and len({m.tobytes() for m in moved}) > 3, r
    ctx = b.Context(b.make_config(B, T, k, 4, 32, k, H, latent_fmt=fmt, slots_per_seq=k, sm_scale=scale))
    out = torch.empty((B, T, H, 512), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((B, T, H), dtype=torch.float32, device="cuda")
    ctx.sparse_mla_decode(q.cuda(), pool.cuda(), torch.from_numpy(idx).cuda(), out, lse)
    torch.cuda.synchronize()
    ro, rl = O.sparse_mla(_qbits(q), pool.numpy(), idx, fmt, scale)
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - ro) <= 1e-2 * np.linalg.norm(ro)
    assert np.allclose(lse.cpu().numpy(), rl, atol=1e-3 * max(scale, 1.0), rtol=1e-5)
    ctx.close()


@pytest.mark.parametrize("fmt,B,T,H,k", [(0, 12, 1, 128, 256), (1, 6, 2, 40, 256), (0, 7, 2, 33, 300), (1, 33, 1, 16, 128), (0, 4, 1, 128, 320)])
def test_offloaded_rows_finished_by_attn1(ess_lib, fmt, B, T, H, k):
    """Twelve rows and more: Attn1 merges the partial results of Attn0 (one to eight ranges) in its epilogue; fewer: both
    lists in one form of the kernel.  Steps in which everything misses (Attn0 has nothing), some and nothing misses
    (Attn1 has nothing), against the oracle; every schedule gives the same bits."""
    from paper_2512_10576_amd import binding as b
    print("finished by attn1", fmt, B, T, H, k, flush=True)
    L, S = 2048, 1024
    stride = (1152, 656)[fmt]
    host = (synth.latent_rows_bf16, synth.latent_rows_fp8)[fmt](11, B * L).reshape(B, L, stride)
    hp = torch.empty((B, L, stride), dtype=torch.uint8, pin_memory=True)
    hp.copy_(host)
    qi, w, key = synth.indexer_inputs(5, B, T, 4, 32, L, 4, 4, 8)
    rng = np.random.default_rng(B + k)
    first = np.stack([rng.permutation(L)[:k] for _ in range(B * T)]).astype(np.int32).reshape(B, T, k)
    some = first.copy()
    for r, row in enumerate(some.reshape(B * T, k)):
        n = (1, k // 2, k - 1, 0)[r % 4]
        row[:n] = rng.permutation(L)[:n]
        row[:] = rng.permutation(row)                             # duplicates within a list never occur in a selection
        if len(set(row.tolist())) < k:
            row[:] = rng.permutation(L)[:k]
    sets = [np.sort(x, axis=2) for x in (first, some, some)]
    runs = {}
    for flags in (0, b.ESS_FLAG_SERIAL, b.ESS_FLAG_DBA, b.ESS_FLAG_AUTO):
        ctx = b.Context(b.make_config(B, T, L, 4, 32, k, H, latent_fmt=fmt, slots_per_seq=S, flags=flags))
        cache = b.Cache.allocate(ctx.cfg, B, host_pool=hp)
        ctx.cache_reset(cache, B)
        oc, opool = O.SlotCache(B, L, S), np.zeros((B, S, stride), np.uint8)
        lens = torch.full((B,), L, dtype=torch.int32)
        got = []
        for step, sel in enumerate(sets, 1):
            q = synth.attn_query(60 + step, B, T, H)
            idx = torch.empty((B, T, k), dtype=torch.int32, device="cuda")
            out = torch.full((B, T, H, 512), 9.0, dtype=torch.bfloat16, device="cuda")
            lse = torch.full((B, T, H), 9.0, dtype=torch.float32, device="cuda")
            ctx.decode_step(cache, qi.cuda(), w.cuda(), key.cuda(), lens.cuda(), q.cuda(), step, idx, out, lse, None, torch.from_numpy(sel).cuda())
            torch.cuda.synchronize()
            if flags == 0:
                r = O.decode_step(qi.numpy(), w.numpy(), key.numpy(), lens.numpy(), k, oc, opool, host.numpy(), _qbits(q), fmt,
                                  576 ** -0.5, step, sel)
                # Attn0 of twelve rows and more dequantises to bf16: an entry's logit, of standard deviation 1, is off by
                # 2^-9 / sqrt(3) = 1.1e-3 of it (standard deviation), a log-sum-exp over several hundred by a part of that
                _check(out, lse, r["out"], r["lse"], 2e-3 if fmt and B * T >= 12 else 1e-4)
            got.append((out, lse))
        runs[flags] = got
        ctx.close()
    for flags, got in runs.items():
        for (o0, l0), (o1, l1) in zip(runs[0], got):
            assert torch.equal(o0, o1) and torch.equal(l0, l1), flags


@pytest.mark.parametrize("H,k", [(128, 64), (40, 640), (128, 2048), (128, 2100)])
def test_values_beyond_fp16_in_every_form(ess_lib, H, k):
    """One row: finished by the kernel of 32 heads (64 entries), several ranges of it (640, 2048), and the kernel of 128 heads.
    With all logits equal the output is the entry itself, exactly, for values within 2^29 of a head's largest one; a value
    2^81 below it is exact or zero."""
    from paper_2512_10576_amd import binding as b
    print("values beyond fp16", H, k, flush=True)
    vals = {0: 1.0e30, 1: -7.5e29, 2: 9.5e23, 3: 3.0e5, 200: 2.5e29, 511: -1.0e30}
    rows = torch.zeros((1, k, 576), dtype=torch.bfloat16)
    for col, v in vals.items():
        rows[..., col] = v
    ctx = b.Context(b.make_config(1, 1, k, 4, 32, k, H, slots_per_seq=k))
    out = torch.full((1, 1, H, 512), 9.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, 1, H), 9.0, dtype=torch.float32, device="cuda")
    idx = torch.arange(k, dtype=torch.int32, device="cuda").view(1, 1, k)
    ctx.sparse_mla_decode(torch.zeros((1, 1, H, 576), dtype=torch.bfloat16, device="cuda"), rows.view(torch.uint8).reshape(1, k, 1152).cuda(), idx, out, lse)
    torch.cuda.synchronize()
    got, want = out.float().cpu()[0, 0], rows[0, 0, :512].float()
    keep = [c for c in range(512) if c != 3]
    assert torch.equal(got[:, keep], want[keep].expand(H, -1))
    assert bool(((got[:, 3] == 0) | (got[:, 3] == want[3])).all())
    assert np.allclose(lse.cpu().numpy(), np.log(k), atol=1e-4)
    ctx.close()
