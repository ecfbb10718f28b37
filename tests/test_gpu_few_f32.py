"""fp32 steps whose workgroups deal the keys of one 32-row unit to their wavefronts: every row against the oracle, with the launch plan's
own choice, which is checked to be this kernel's."""
import pytest
import torch

import paper_2605_12471_amd as kv
from paper_2605_12471_amd import binding
from paper_2605_12471_amd import inputs as I
import test_gpu_f32_terms as terms
from test_gpu_parity_small import H, _run_case  # noqa: F401  (H: the fixture)
from test_gpu_window import _run_window_case

pytestmark = pytest.mark.gpu


def _one_unit_workgroups(Hq, Hkv, d, chunks, window=None):
    """Which of the steps have one workgroup per unit and piece (the general kernel's have four units or eight; steps of one unit are not
    told apart)."""
    cfg = binding.make_config(1, Hq, Hkv, d, max(chunks), sum(chunks), kv.KVFOLD_F32)
    pos, got = 0, []
    for n in chunks:
        rc, pl = kv.kvfold_plan_for(cfg, 256, n, pos + n, *(window or (0, 0)))
        assert rc == 0
        units = -(-n * (Hq // Hkv) // 32)
        got.append(pl.n_workgroups == Hkv * units * pl.n_splits and units > 1)
        pos += n
    return got


# The old cache's end before, on and behind every edge of a 32-key block; units that fill and straddle tokens; the last unit with one
# row to 32; pieces that end before the chunk, inside it and behind it; more chunk rows than a workgroup copies in a turn.
@pytest.mark.parametrize("Hq,Hkv,d,chunks", [
    (8, 2, 128, [33, 31, 32, 9, 23, 64, 65, 127, 40]),
    (8, 2, 64, [33, 31, 32, 9, 23, 64, 65, 127, 40]),
    (7, 1, 128, [37, 5, 64, 300, 41, 100]),
    (28, 4, 128, [500, 37, 1, 30]),
    (3, 3, 64, [65, 33, 97, 1000, 34]),
    (40, 1, 128, [1, 2, 61, 3, 50]),
    (32, 8, 128, [1100, 37, 10, 1]),
    (4, 1, 64, [1, 400, 157, 1]),
])
def test_edges_of_blocks_units_and_the_chunk(H, oracle, Hq, Hkv, d, chunks):
    cfg = I.FoldConfig("few_f32", 80, 1, Hq, Hkv, d, max(chunks), 0, "f32")
    assert sum(_one_unit_workgroups(Hq, Hkv, d, chunks)) >= len(chunks) // 2
    _run_case(H, oracle, cfg, chunks)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_sink,window", [(4, 100), (0, 64), (4, 1), (70, 50), (0, 1), (33, 31), (4, 5000)])
def test_windows(H, oracle, d, n_sink, window):
    """Windows shorter than a block and longer than the cache, sinks across two tiles, one row to several units."""
    chunks = [100, 1, 7, 40, 65, 96, 33]
    cfg = I.FoldConfig("few_f32_win", 81, 1, 8, 2, d, max(chunks), 0, "f32")
    assert sum(_one_unit_workgroups(8, 2, d, chunks, (n_sink, window))) >= 3
    _run_window_case(H, oracle, cfg, chunks, n_sink, window)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,hq,hkv,check", [
    (150, 4, 2, lambda d: terms.test_values_that_are_not_finite(d, 0, 0)),
    (70, 4, 2, lambda d: terms.test_finite_values_whose_product_overflows(d, 0)),
    (100, 4, 2, lambda d: terms.test_smallest_values_keep_their_bits(d, 0)),
    (200, 4, 1, lambda d: terms.test_values_over_many_powers_of_two(d, 0)),
    (64, 8, 8, lambda d: terms.test_single_products_are_rounded_once(d, 0)),
])
def test_numbers_that_the_terms_can_and_cannot_hold(d, n, hq, hkv, check):
    """The general kernel's tests of its operands' range, with the plan's own choice."""
    assert _one_unit_workgroups(hq, hkv, d, [n]) == [True]
    check(d)


@pytest.mark.parametrize("d", [64, 128])
def test_rows_beyond_the_terms_with_the_rotary_embedding_and_under_a_window(H, oracle, d):
    """The same for the fp32 instructions' own rotation of the queries, for a window that passes over such a value, and for rows that do not see
    a key that is not finite."""
    assert _one_unit_workgroups(4, 2, d, [100]) == [True]
    terms.test_values_and_queries_beyond_the_terms_with_the_rotary_embedding(H, oracle, d, 0)
    assert _one_unit_workgroups(4, 2, d, [300], (2, 40)) == [True]
    terms.test_values_beyond_the_terms_under_a_window(H, oracle, d, 0, 0)
    assert _one_unit_workgroups(4, 2, d, [200]) == [True]
    terms.test_rows_do_not_notice_what_they_do_not_see(d, 0, 0)


@pytest.mark.parametrize("d", [64, 128])
def test_more_blocks_with_odd_keys_than_a_wavefront_lists(H, d):
    """A value beyond the terms' range in every block of 32 keys: the whole piece goes through the fp32 instructions.  Column 5 of the output is
    2^100 times the weight of these keys together, against 64 bits; the other columns keep their tolerance."""
    h, n, prev = 256, 1, 36 * 32 * (8 if d == 64 else 4)  # one workgroup a head: 36 blocks a wavefront
    rc, pl = kv.kvfold_plan_for(binding.make_config(1, h, h, d, 64, prev + n, kv.KVFOLD_F32), 256, n, prev + n)
    assert rc == 0 and pl.n_splits == 1 and pl.n_workgroups == h
    cfg = I.FoldConfig("few_f32_odd", 82, 1, h, h, d, n, 0, "f32")
    outs = []
    q, k, v = I.chunk_qkv(cfg, 0, 0, n_tokens=n, token_base=0)
    for odd in (False, True):
        gpu = H.GpuFold(cfg, capacity=prev + n, chunk_tokens=64)
        K, V = gpu.cache.view(0)
        for t, part in ((K, 1), (V, 2)):
            t[:, :prev].copy_(terms._random(prev, h, d, part).transpose(0, 1))
        if odd:
            V[:, 0:prev:32, 5] = 2.0 ** 100
        gpu.cache.set_length(-1, prev)
        outs.append(gpu.step(0, q, k, v).cpu().double())
        logits = torch.cat([(K[:, :prev].double() @ q[0].cuda().double()[..., None])[..., 0].cpu(), (q[0].double() * k[0].double()).sum(-1, keepdim=True)], 1)
        gpu.close()
    plain, with_odd = outs
    rest = [c for c in range(d) if c != 5]
    assert (with_odd - plain)[..., rest].abs().max() <= 1e-5
    weights = torch.softmax(logits / d ** 0.5, 1)
    share = with_odd[0, :, 5] / 2.0 ** 100  # (the other keys' values are 2^-100 of it)
    assert (share / weights[:, 0:prev:32].sum(1) - 1.0).abs().max() <= 1e-5  # (the mode's tolerance)
