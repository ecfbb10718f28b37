"""Steps of at most 32 packed rows per KV head (decoding): every row against the oracle around the 32-key block and the
64-key tile, with and without a split, and against the general kernel where the oracle has no answer."""
import math

import pytest
import torch

import paper_2605_12471_amd as kv
from paper_2605_12471_amd import inputs as I
from test_gpu_parity_small import H, _run_case  # noqa: F401  (H: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,Hkv", [(1, 3), (3, 2), (4, 2), (7, 1), (32, 1)])
@pytest.mark.parametrize("splits", [0, 1, 2, 5])
def test_edges_of_blocks_tiles_and_rows(H, oracle, d, G, Hkv, splits):
    """From an empty cache on: lengths that straddle, meet and pass the edges of blocks and tiles, one row to 32."""
    n = 32 // G
    cfg = I.FoldConfig("few", 65, 1, G * Hkv, Hkv, d, 200, 0, "bf16")
    _run_case(H, oracle, cfg, [1, n, 31, 1, n, 61 - n, 1, 1, 200, n, 1, max(1, n - 1), 1], splits=splits)


@pytest.mark.parametrize("G,d", [(16, 128), (17, 128), (16, 64), (17, 64)])
def test_sixteen_rows_and_more(H, oracle, G, d):
    """16 rows of 128 columns and 32 of 64 have their keys straight from memory; a wavefront's blocks from none to a handful, odd and
    even numbers, the last one with rows of the chunk, beyond it, or neither."""
    cfg = I.FoldConfig("few16", 67, 1, G, 1, d, 160, 0, "bf16")
    _run_case(H, oracle, cfg, [1, 1, 30, 1, 95, 1, 1, 127, 1, 160, 1, 94, 1, 1], splits=1)


@pytest.mark.parametrize("profile", sorted(I.LOGIT_PROFILES))
def test_logit_jumps(H, oracle, profile):
    cfg = I.FoldConfig("few_jump", 66, 1, 4, 1, 128, 400, 0, "bf16")
    _run_case(H, oracle, cfg, [400, 8, 1, 7], profile=profile, check_lse=False)


def _filled(Hq, Hkv, d, n, L):
    g = torch.Generator("cuda").manual_seed(L)
    cache = kv.KvFoldCache(1, Hq, Hkv, d, n, L + n, "bf16")
    for rows in cache.view(0):
        rows[:, :L].normal_(generator=g)
    cache.set_length(-1, L)
    return cache, [torch.randn(n, h, d, generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv)]


def _step(cache, L, args, **kw):
    out = torch.full_like(args[0], 7.0)
    cache.set_length(0, L)
    cache.step(0, *args, out, pos_offset=L, **kw)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("splits", [1, 4])
def test_append_inside_or_before(splits):
    """The same bits, outputs and cache rows, whether the kernel appends by itself or reads rows appended before."""
    L, n = 1000 + 13, 8
    cache, args = _filled(8, 2, 128, n, L)
    cache.set_tuning(kv.TUNE_SPLITS, splits)
    one = _step(cache, L, args)
    rows = [t[:, L:L + n].clone() for t in cache.view(0)]
    for t in cache.view(0):
        t[:, L:L + n] = 0
    cache.set_tuning(kv.TUNE_FUSED_APPEND, 1)
    assert torch.equal(one, _step(cache, L, args))
    for t, r, new in zip(cache.view(0), rows, args[1:]):
        assert torch.equal(t[:, L:L + n], r) and torch.equal(r, new.transpose(0, 1))
    cache.close()


@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("d", [64, 128])
def test_values_that_are_not_finite(d, splits):
    """Not a number where the general kernel has none, infinite where it is, equal to rounding elsewhere: an infinite and a
    NaN value, a key at -inf, a NaN key, a NaN query."""
    L, n = 700, 4
    cache, args = _filled(16, 4, d, n, L)
    K, V = cache.view(0)
    args[0][:, :4, 3] = -args[0][:, :4, 3].abs() - 0.1  # KV head 0: its queries see key 40 at -inf
    K[0, 40, 3] = math.inf
    V[1, 300, 5] = math.inf
    V[1, 301, 6] = math.nan
    K[2, 500, 0] = math.nan
    args[0][2, 13] = math.nan
    cache.set_tuning(kv.TUNE_SPLITS, splits)
    got = _step(cache, L, args).float()
    cache.set_tuning(kv.TUNE_UNITS_PER_WAVE, 1)
    want = _step(cache, L, args).float()
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isinf(got), torch.isinf(want))
    assert torch.isnan(got[:, 8:12]).all() and torch.isinf(got[:, 4:8, 5]).all() and torch.isfinite(got[:, :4]).all()
    ok = torch.isfinite(want)
    # each is a sum of values below 5 with weights rounded to 2^-9 and an output rounded to 2^-9 of its size
    assert (got - want)[ok].abs().max() <= 2e-2
    cache.close()


def test_graph_replays():
    L = 5000
    cache, args = _filled(32, 8, 128, 1, L)
    want = _step(cache, L, args)
    out = torch.empty_like(want)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    cache.set_length(0, L)
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            cache.step(0, *args, out, pos_offset=L)
    torch.cuda.synchronize()
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(_step(cache, L, args), want)
    cache.close()


def test_cache_created_while_a_stream_is_captured():
    """Creating a cache touches no other stream: not the legacy one, which a capture in relaxed mode would not survive.  With the static
    counters all taken, so that it clears counters of its own."""
    L = 1000
    cache, args = _filled(8, 2, 128, 1, L)
    holders = [kv.KvFoldCache(1, 8, 2, 128, 1, L + 1, "bf16") for _ in range(64)]
    want = _step(cache, L, args)
    out = torch.zeros_like(want)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    cache.set_length(0, L)
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side, capture_error_mode="relaxed"):
            other = kv.KvFoldCache(1, 8, 2, 128, 1, L + 1, "bf16")
            cache.step(0, *args, out, pos_offset=L)
    torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    for rows, filled in zip(other.view(0), cache.view(0)):
        rows.copy_(filled)
    other.set_length(0, L)
    assert torch.equal(_step(other, L, args), want)
    for c in [other, cache] + holders:
        c.close()


def test_counters_of_many_caches():
    """More caches than there are static counters, some given back in between: the same bits from each.  (Whose counters are whose: the host model.)"""
    L = 1000
    first, args = _filled(8, 2, 128, 1, L)
    want = _step(first, L, args)
    caches = [_filled(8, 2, 128, 1, L)[0] for _ in range(70)]
    assert all(torch.equal(_step(c, L, args), want) for c in caches for _ in range(2))
    for c in caches[10:30] + [first]:
        c.close()
    again = [_filled(8, 2, 128, 1, L)[0] for _ in range(3)]
    for c in caches[:10] + again + caches[30:]:
        assert torch.equal(_step(c, L, args), want)
        c.close()


def _by_merge_kernel(cache, L, args, **kw):
    """The step with its pieces merged by the merge kernel: the output's first row lies on the last row's last query."""
    q = args[0]
    both = torch.zeros(2 * q.numel(), device="cuda", dtype=q.dtype)
    out = both[q.numel() - 8:2 * q.numel() - 8].view(q.shape)
    cache.set_length(0, L)
    cache.profile_begin(1)
    cache.step(0, both[:q.numel()].view(q.shape).copy_(q), *args[1:], out, pos_offset=L, **kw)
    assert cache.profile_end()[3] > 0
    return out.clone()


def _in_the_kernel(cache, L, args, **kw):
    """The step with pieces that meet in the attention kernel, and no append kernel in front."""
    cache.profile_begin(1)
    out = _step(cache, L, args, **kw)
    _, append_ms, _, merge_ms = cache.profile_end()
    assert append_ms == 0 and merge_ms == 0
    return out


@pytest.mark.parametrize("Hq,Hkv,d,n", [(2, 2, 128, 4), (8, 2, 128, 2), (2, 2, 64, 4), (8, 2, 64, 2)])
def test_pieces_of_which_a_row_sees_nothing(Hq, Hkv, d, n):
    """Pieces of a tile each, the chunk's first row the last key of the last but one: the first token sees nothing of the last piece, whose values are NaN
    and infinite.  One row sees every key of every piece at -inf.  One row of a wavefront and two."""
    L = 64 * 5 - 1
    cache, (q, k, v) = _filled(Hq, Hkv, d, n, L)
    v[1:, 0], v[1:, 1, 5] = math.nan, math.inf
    for rows in (cache.view(0)[0][-1, :L], k[:, -1]):
        rows[:, 3] = 3e38
    q[:, -(Hq // Hkv):, 3] = 0
    q[0, -1, 3] = -3e38
    cache.set_tuning(kv.TUNE_SPLITS, 6)
    assert cache.plan(n, L + n)[1] == 6
    lse = torch.zeros(Hq, n, device="cuda")
    got = _in_the_kernel(cache, L, (q, k, v), lse=lse).float()
    want = _by_merge_kernel(cache, L, (q, k, v)).float()
    assert torch.isfinite(got[0, :-1]).all() and torch.isnan(got[0, -1]).all()
    assert torch.isnan(got[1:, :Hq // Hkv]).all() and not torch.isfinite(got[1:, -(Hq // Hkv):, 5]).any()
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isinf(got), torch.isinf(want))
    ok = torch.isfinite(want)
    assert ((got - want)[ok].abs() <= 2.0 ** -7 * want[ok].abs() + 1e-6).all()  # (sums in another order: neighbours at most)
    assert lse[-1, 0] == -math.inf and torch.isfinite(lse.flatten()[torch.arange(Hq * n) != (Hq - 1) * n]).all()
    cache.close()


@pytest.mark.parametrize("Hq,Hkv,d,n", [(32, 8, 128, 1), (8, 2, 128, 2), (4, 4, 64, 4), (16, 2, 64, 1)])
@pytest.mark.parametrize("bits,rope", [(0, True), (8, False), (4, True)])
@pytest.mark.parametrize("L", [700, 64 * 11 - 1])
def test_pieces_that_meet_and_rows_that_their_readers_work_on(Hq, Hkv, d, n, bits, rope, L):
    """The rotary embedding and the round trip inside a step whose pieces meet: the bits, outputs and cache rows, of the step behind an append kernel, and
    within rounding those of the merge kernel."""
    cache, args = _filled(Hq, Hkv, d, n, L)
    cache.set_storage_roundtrip(bits)
    cache.set_tuning(kv.TUNE_SPLITS, 6)
    kw = {"rope": I.rope_tables(d, L, n, device="cuda")} if rope else {}
    one = _in_the_kernel(cache, L, args, **kw)
    rows = [t[:, L:L + n].clone() for t in cache.view(0)]
    for t in cache.view(0):
        t[:, L:L + n] = 0
    want = _by_merge_kernel(cache, L, args, **kw).float()
    assert ((one.float() - want).abs() <= 2.0 ** -7 * want.abs() + 1e-6).all()
    assert all(torch.equal(t[:, L:L + n], r) for t, r in zip(cache.view(0), rows))
    cache.set_tuning(kv.TUNE_FUSED_APPEND, 1)
    for t in cache.view(0):
        t[:, L:L + n] = 0
    assert torch.equal(one, _step(cache, L, args, **kw))
    assert all(torch.equal(t[:, L:L + n], r) for t, r in zip(cache.view(0), rows))
    cache.close()


@pytest.mark.parametrize("Hq,Hkv,d,n", [(32, 8, 128, 1), (8, 2, 64, 1), (3, 3, 128, 4), (2, 2, 64, 1), (10, 2, 128, 1), (8, 1, 64, 1), (7, 1, 128, 1), (9, 1, 64, 1)])
@pytest.mark.parametrize("splits,tiles", [(2, 22), (6, 22), (7, 21), (12, 24), (13, 26), (24, 24), (25, 25), (32, 32), (33, 33)])
def test_pieces_that_meet_in_the_last_workgroup(Hq, Hkv, d, n, splits, tiles):
    """Up to eight rows and 32 pieces (128 wide, more than four rows: twelve): a lane's six, and more, a row of a wavefront or two, and the merge kernel beyond, with piece counts that change
    from step to step; within the rounding of the output, and the same bits every time, wherever the partial results lie."""
    L = 64 * (tiles - 1) + 17
    cache, args = _filled(Hq, Hkv, d, n, L)
    cache.set_tuning(kv.TUNE_SPLITS, splits)
    want = _by_merge_kernel(cache, L, args).float()
    lse = [torch.empty(Hq, n, device="cuda") for _ in range(2)]
    assert cache.plan(n, L + n)[1] == splits
    cache.profile_begin(1)
    one = _step(cache, L, args, lse=lse[0])
    rows = n * Hq // Hkv
    assert (cache.profile_end()[3] > 0) == (rows > 8 or splits > (32 if d == 64 or rows <= 4 else 12))
    assert torch.equal(one, _step(cache, L, args, noalloc=True))
    # the sums differ in fp32's last places, so that the outputs are equal or neighbours, and those are at most 2^-7 of the value apart
    assert ((one.float() - want).abs() <= 2.0 ** -7 * want.abs() + 1e-6).all()
    for other in (3, tiles, splits, 11):
        cache.set_tuning(kv.TUNE_SPLITS, other)
        again = _step(cache, L, args, lse=lse[1])
        if other == splits:
            assert torch.equal(one, again) and torch.equal(*lse)
    cache.set_tuning(kv.TUNE_SPLITS, 1)
    _step(cache, L, args, lse=lse[1])
    assert (lse[0] - lse[1]).abs().max() <= 1e-4
    cache.close()


@pytest.mark.parametrize("on", ["k", "v", "q", "next"])
def test_pieces_that_meet_under_an_output_on_the_inputs(on):
    """The output on rows that other heads' workgroups still read -- new rows, or other rows' queries -- has the same bits."""
    Hq, Hkv, d, n, L = 64, 32, 128, 2, 900
    cache, (q, k, v) = _filled(Hq, Hkv, d, n, L)
    cache.set_tuning(kv.TUNE_SPLITS, 3)
    want = _step(cache, L, (q, k, v))
    rows = [t[:, L:L + n].clone() for t in cache.view(0)]
    for _ in range(5):
        both = torch.zeros(2 * q.numel(), device="cuda", dtype=torch.bfloat16)
        at = {"next": d}.get(on, 0)
        src = {"k": k, "v": v}.get(on, q)
        put = both[:src.numel()].view(src.shape)
        put.copy_(src)
        args = {"k": (q, put, v), "v": (q, k, put)}.get(on, (put, k, v))
        out = both[at:at + q.numel()].view(q.shape)
        for t in cache.view(0):
            t[:, L:L + n] = 0
        cache.set_length(0, L)
        cache.step(0, *args, out, pos_offset=L)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert all(torch.equal(t[:, L:L + n], r) for t, r in zip(cache.view(0), rows))
    cache.close()
