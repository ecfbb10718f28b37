"""The merge of split steps: a piece in which a row sees no key leaves the row as it is."""
import math

import pytest
import torch

import paper_2605_12471_amd as kv
from paper_2605_12471_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    from tests import fold_harness
    return fold_harness


# Two pieces that meet at key 64, one head per group, 48 keys before the chunk: row i stands at position 48 + i, so that the edge lies inside
# a unit of 32 rows.  Without a window rows 0 .. 15 see nothing of the second piece, where key 70 lies; with one of 32 keys, rows
# from 47 on see nothing of the first, where key 20 lies.  More pieces than a thread of the merge has in one LDS group: long prefix.
@pytest.mark.parametrize("bad", [math.inf, math.nan])
@pytest.mark.parametrize("dtype,d,prev,n,upw,splits,window,key,clean", [
    ("f32", 128, 48, 32, 1, 2, None, 70, slice(0, 16)),
    ("f32", 64, 48, 80, 2, 2, None, 70, slice(0, 16)),
    ("bf16", 128, 48, 32, 0, 2, None, 70, slice(0, 16)),   # the kernel for few rows
    ("bf16", 64, 48, 32, 0, 2, None, 70, slice(0, 16)),
    ("bf16", 128, 48, 64, 1, 2, None, 70, slice(0, 16)),
    ("bf16", 64, 48, 64, 2, 2, None, 70, slice(0, 16)),
    ("bf16", 128, 48, 72, 2, 2, None, 70, slice(0, 16)),
    ("bf16", 128, 48, 64, 1, 2, (0, 32), 20, slice(47, 64)),
    ("f32", 128, 48, 64, 1, 2, (0, 32), 20, slice(47, 64)),
    ("bf16", 128, 1200, 64, 1, 20, None, 1223, slice(0, 16)),
    ("f32", 128, 1200, 64, 1, 20, None, 1223, slice(0, 16)),
])
def test_a_value_that_a_row_does_not_see_leaves_it_as_it_is(H, dtype, d, prev, n, upw, splits, window, key, clean, bad):
    cfg = I.FoldConfig("merge", 31, 1, 2, 2, d, max(prev, n), 0, dtype)
    res = []
    for value in (1.0, bad):
        gpu = H.GpuFold(cfg, capacity=prev + n, chunk_tokens=max(prev, n))
        gpu.cache.set_tuning(kv.TUNE_UNITS_PER_WAVE, upw)
        pos = 0
        for step, C in enumerate((prev, n)):
            gpu.cache.set_tuning(kv.TUNE_SPLITS, splits if step else 1)
            q, k, v = I.chunk_qkv(cfg, 0, step, n_tokens=C, token_base=pos)
            if pos <= key < pos + C:
                v[key - pos, :, 3] = value
            if step:
                assert gpu.cache.plan(n, prev + n)[1] == splits
            out, lse = gpu.step(0, q, k, v, want_lse=True, **({"window": window} if window and step else {}))
            pos += C
        res.append((out.clone(), lse.clone()))
        gpu.close()
    (plain, plain_lse), (out, lse) = res
    assert torch.isfinite(plain).all() and not torch.isfinite(out).all()
    assert torch.equal(out[clean], plain[clean]) and torch.equal(lse[:, clean], plain_lse[:, clean])


@pytest.mark.parametrize("dtype,d,n,upw", [("f32", 128, 40, 1), ("f32", 64, 72, 2), ("bf16", 128, 16, 0), ("bf16", 64, 40, 1), ("bf16", 128, 72, 2)])
@pytest.mark.parametrize("splits", [1, 2, 20])
def test_rows_whose_every_key_is_hidden(H, dtype, d, n, upw, splits):
    """A query with -inf where every key is positive: all its logits are -inf, the log-sum-exp too, and there is no output; the other rows
    keep their bits."""
    prev = 1200
    cfg = I.FoldConfig("hidden", 32, 1, 2, 2, d, prev, 0, dtype)
    res = []
    for value in (0.0, -math.inf):
        gpu = H.GpuFold(cfg, capacity=prev + n, chunk_tokens=prev)
        gpu.cache.set_tuning(kv.TUNE_UNITS_PER_WAVE, upw)
        pos = 0
        for step, C in enumerate((prev, n)):
            gpu.cache.set_tuning(kv.TUNE_SPLITS, splits if step else 1)
            q, k, v = I.chunk_qkv(cfg, 0, step, n_tokens=C, token_base=pos)
            k[:, :, 5] = 1.0
            if step:
                q[3::7, :, 5] = value
                assert gpu.cache.plan(n, prev + n)[1] in (splits, 19)  # (16 tokens have 19 tiles of keys)
            out, lse = gpu.step(0, q, k, v, want_lse=True)
            pos += C
        res.append((out.clone(), lse.clone()))
        gpu.close()
    (plain, plain_lse), (out, lse) = res
    hidden = torch.zeros(n, dtype=torch.bool, device="cuda")
    hidden[3::7] = True
    assert torch.isfinite(plain).all() and torch.isfinite(plain_lse).all()
    assert torch.isnan(out[hidden]).all() and (lse[:, hidden] == -math.inf).all()
    assert torch.equal(out[~hidden], plain[~hidden]) and torch.equal(lse[:, ~hidden], plain_lse[:, ~hidden])


# Rows that fill their blocks and leave some over, blocks that are a multiple of the XCDs' number and not, one split group per row up to eight.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 7, 37, 150, 1030])
@pytest.mark.parametrize("splits", [2, 9, 18])
def test_every_row_comes_out_in_its_place(H, d, n, splits):
    """Against the unsplit step.  Both hold the sums in fp32, in another order: at most 1200 + n terms in 64-key tiles of a 16-long
    chain, |v| < 6, so some 100 roundings of 2^-24 each."""
    prev = 1200
    cfg = I.FoldConfig("rows", 33, 1, 2, 1, d, prev, 0, "f32")
    res = []
    for s in (1, splits):
        gpu = H.GpuFold(cfg, capacity=prev + n, chunk_tokens=prev)
        pos = 0
        for step, C in enumerate((prev, n)):
            gpu.cache.set_tuning(kv.TUNE_SPLITS, s if step else 1)
            q, k, v = I.chunk_qkv(cfg, 0, step, n_tokens=C, token_base=pos)
            out, lse = gpu.step(0, q, k, v, want_lse=True)
            pos += C
        assert s / 2 < gpu.cache.plan(n, prev + n)[1] <= s  # (whole tiles)
        res.append((out.clone(), lse.clone()))
        gpu.close()
    assert (res[0][0] - res[1][0]).abs().max() <= 100 * 2.0 ** -24 * 6
    assert (res[0][1] - res[1][1]).abs().max() <= 100 * 2.0 ** -24 * 16


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("upw", [1, 2])
@pytest.mark.parametrize("n", [9, 33, 64, 300])
def test_two_pieces_meet_in_the_attention_kernel(H, d, upw, n):
    """The bits are the merge kernel's (an output on other rows' queries sends the step there), step after step with whatever counts lie
    between: partly filled units, wavefronts without rows, a later piece with little in it; with the output in the place of the queries, and
    with the partial results in static scratch."""
    Hq, Hkv, prev = 8, 2, 700
    g = torch.Generator("cuda").manual_seed(n + d)
    q, k, v = (torch.randn(n, h, d, generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    cache = kv.KvFoldCache(1, Hq, Hkv, d, 300, prev + n, "bf16")
    for rows in cache.view(0):
        rows[:, :prev].normal_(generator=g)
    cache.set_tuning(kv.TUNE_UNITS_PER_WAVE, upw)
    cache.set_tuning(kv.TUNE_SPLITS, 2)

    def step(q, out, merge=False, **kw):
        lse = torch.empty(Hq, n, device="cuda")
        cache.set_length(0, prev)
        cache.profile_begin(1)
        cache.step(0, q, k, v, out, pos_offset=prev, lse=lse, **kw)
        assert (cache.profile_end()[3] > 0) == merge
        return out.clone(), lse
    both = torch.empty(q.numel() + Hq * d, device="cuda", dtype=torch.bfloat16)
    at = both[:q.numel()].view(q.shape)
    want = step(at.copy_(q), both[Hq * d:].view(q.shape), merge=True)  # the output one token further on
    for _ in range(3):
        assert all(torch.equal(a, b) for a, b in zip(want, step(q, torch.full_like(q, 7.0))))
    assert all(torch.equal(a, b) for a, b in zip(want, step(q, torch.full_like(q, 7.0), noalloc=True)))
    assert all(torch.equal(a, b) for a, b in zip(want, step(at.copy_(q), at)))
    assert all(torch.equal(a, b) for a, b in zip(want, step(at.copy_(q), both[Hq * d:].view(q.shape), merge=True)))
    assert all(torch.equal(a, b) for a, b in zip(want, step(q, torch.empty_like(q))))
    cache.close()


@pytest.mark.parametrize("n,splits", [(1, 4), (2, 3), (64, 2)])
@pytest.mark.parametrize("on", ["cos", "sin", "keys", "values", "lse on keys", "lse on cos"])
def test_results_on_what_other_workgroups_still_read(n, splits, on):
    """Pieces that meet in the attention kernel store results while other workgroups read the angles and the cached rows: results that lie on
    these go through the merge kernel, with the bits of one on other rows' queries, which has always done so."""
    Hq, Hkv, d, prev = 64, 32, 128, 900
    g = torch.Generator("cuda").manual_seed(n)
    q, k, v = (torch.randn(n, h, d, generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    tables = I.rope_tables(d, prev, n, device="cuda")
    cache = kv.KvFoldCache(1, Hq, Hkv, d, 256, 1024, "bf16")
    if n > 8:
        cache.set_tuning(kv.TUNE_UNITS_PER_WAVE, 1)
    cache.set_tuning(kv.TUNE_SPLITS, splits)
    filled = [torch.randn(Hkv, prev, d, generator=g, device="cuda").bfloat16() for _ in range(2)]

    def step(out, lse, rope, q=q):
        for rows, values in zip(cache.view(0), filled):
            rows[:, :prev] = values
        cache.set_length(0, prev)
        torch.cuda.synchronize()
        cache.profile_begin(1)
        cache.step(0, q, k, v, out, pos_offset=prev, lse=lse, rope=rope)
        merge_ms = cache.profile_end()[3]
        return out.clone(), lse.clone(), merge_ms > 0
    assert not step(torch.empty_like(q), torch.empty(Hq, n, device="cuda"), tables)[2]
    both = torch.zeros(2 * q.numel(), device="cuda", dtype=q.dtype)
    want = step(both[q.numel() - 8:-8].view(q.shape), torch.empty(Hq, n, device="cuda"), tables, both[:q.numel()].view(q.shape).copy_(q))
    assert want[2]
    for _ in range(3):
        room = torch.zeros(max(q.numel() // 2, n * d), device="cuda")  # floats
        rope, out, lse = tables, torch.empty_like(q), torch.empty(Hq, n, device="cuda")
        if "keys" in on or "values" in on:
            at = cache.view(0)[0 if "keys" in on else 1].reshape(-1)
        else:
            rope = tuple(t if i != on.endswith("sin") else room[:t.numel()].view(t.shape).copy_(t) for i, t in enumerate(tables))
            at = room.view(torch.bfloat16)
        if "lse" in on:
            lse = at[:2 * lse.numel()].view(torch.float32).view(lse.shape)
        else:
            out = at[:q.numel()].view(q.shape)
        got = step(out, lse, rope)
        assert got[2] and torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    cache.close()
