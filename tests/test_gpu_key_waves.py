"""bf16 steps whose workgroups deal the keys of one 32-row unit to their wavefronts, with more than one unit per KV head or under a
window: every row against the oracle, with the launch plan's own choice, which is checked to be this kernel's."""
import pytest

import paper_2605_12471_amd as kv
from paper_2605_12471_amd import binding
from paper_2605_12471_amd import inputs as I
from test_gpu_parity_small import H, _run_case  # noqa: F401  (H: the fixture)
from test_gpu_window import _run_window_case

pytestmark = pytest.mark.gpu


def _one_unit_workgroups(Hq, Hkv, d, chunks, window=None):
    """Which of the steps have one workgroup per unit and piece (the general kernels' have four units or eight)."""
    cfg = binding.make_config(1, Hq, Hkv, d, max(chunks), sum(chunks), kv.KVFOLD_BF16)
    pos, got = 0, []
    for n in chunks:
        rc, pl = kv.kvfold_plan_for(cfg, 256, n, pos + n, *(window or (0, 0)))
        assert rc == 0
        units = -(-n * (Hq // Hkv) // 32)
        got.append(pl.n_workgroups == Hkv * units * pl.n_splits and units > 1)
        pos += n
    return got


# The old cache's end before, on and behind every edge of a 32-key block and a 64-key tile; units that fill and straddle tokens; the last
# unit with one row to 32; pieces that end before the chunk, inside it and behind it; more chunk rows than a workgroup copies in a turn.
@pytest.mark.parametrize("Hq,Hkv,d,chunks", [
    (8, 2, 128, [33, 31, 32, 9, 23, 64, 65, 127, 40]),
    (8, 2, 64, [33, 31, 32, 9, 23, 64, 65, 127, 40]),
    (7, 1, 128, [37, 5, 64, 300, 41, 100]),
    (28, 4, 128, [500, 37, 128, 30]),
    (3, 3, 64, [65, 33, 97, 1000, 34]),
    (40, 1, 128, [1, 2, 61, 3, 200]),
    (32, 8, 128, [1100, 37, 100]),
    (4, 1, 64, [1, 700, 257]),
])
def test_edges_of_blocks_units_and_the_chunk(H, oracle, Hq, Hkv, d, chunks):
    cfg = I.FoldConfig("key_waves", 70, 1, Hq, Hkv, d, max(chunks), 0, "bf16")
    assert sum(_one_unit_workgroups(Hq, Hkv, d, chunks)) >= len(chunks) // 2
    _run_case(H, oracle, cfg, chunks)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_sink,window", [(4, 100), (0, 64), (4, 1), (70, 50), (0, 1), (33, 31), (4, 5000)])
def test_windows(H, oracle, d, n_sink, window):
    """Windows shorter than a block and longer than the cache, sinks across two tiles, one row to several units."""
    chunks = [300, 1, 7, 40, 65, 96, 33]
    cfg = I.FoldConfig("key_waves_win", 71, 1, 8, 2, d, max(chunks), 0, "bf16")
    assert sum(_one_unit_workgroups(8, 2, d, chunks, (n_sink, window))) >= 3
    _run_window_case(H, oracle, cfg, chunks, n_sink, window)


@pytest.mark.parametrize("profile", sorted(I.LOGIT_PROFILES))
def test_logit_jumps(H, oracle, profile):
    chunks = [400, 40, 9, 70]
    cfg = I.FoldConfig("key_waves_jump", 72, 1, 4, 1, 128, 400, 0, "bf16")
    _run_case(H, oracle, cfg, chunks, profile=profile, check_lse=False)


# Blocks that lie in the chunk, before it and on both sides; rows that run past the chunk; the most rows that take this route (100, 64 wide 256)
# and the first that do not; pieces that begin in the chunk.
@pytest.mark.parametrize("Hq,Hkv,d,chunks", [
    (8, 2, 128, [257, 33, 31, 32, 9, 23, 64, 65, 100, 101, 40]),
    (8, 2, 64, [257, 33, 31, 32, 9, 23, 64, 65, 127, 256]),
    (7, 1, 128, [300, 37, 5, 64, 41, 100]),
    (28, 4, 128, [500, 37, 90, 30]),
    (3, 3, 64, [400, 65, 33, 97, 34]),
    (32, 8, 128, [240, 37, 100, 40, 9]),
    (4, 1, 64, [700, 257, 9, 60]),
])
def test_rows_rotated_by_their_readers(H, oracle, Hq, Hkv, d, chunks):
    """Rotary embedding: outputs and cache are the same bits as behind the append kernel (tuning knob), and there is none."""
    cfg = I.FoldConfig("key_waves_rope", 73, 1, Hq, Hkv, d, max(chunks), 0, "bf16")
    own = _one_unit_workgroups(Hq, Hkv, d, chunks)
    takes = [o and n <= (100 if d == 128 else 256) and sum(chunks[:i + 1]) > 256 for i, (o, n) in enumerate(zip(own, chunks))]
    assert sum(takes) >= 2
    res = []
    for knob in (0, 1):
        gpu = H.GpuFold(cfg, capacity=sum(chunks), chunk_tokens=max(chunks))
        gpu.cache.set_tuning(kv.TUNE_FUSED_APPEND, knob)
        outs, pos = [], 0
        for step, C in enumerate(chunks):
            q, k, v = I.chunk_qkv(cfg, 0, step, n_tokens=C, token_base=pos)
            gpu.cache.profile_begin(1)
            outs += list(gpu.step(0, q, k, v, want_lse=True, rope=I.rope_tables(d, pos, C, device="cuda")))
            _, append_ms, _, _ = gpu.cache.profile_end()
            if C * Hq // Hkv > 32:
                assert (append_ms == 0) == (knob == 0 and takes[step])
            pos += C
        K, V = gpu.cache.view(0)
        res.append([*outs, K[:, :pos].clone(), V[:, :pos].clone()])
        gpu.close()
    assert all(bool((a == b).all()) for a, b in zip(*res))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,window,key,blind", [
    (32, None, 47, slice(0, 16)),          # one unit: wavefront 1 has block 1, of which the first 16 rows see nothing
    (64, None, 47, slice(0, 16)),          # several units
    (64, (0, 8), 10, slice(23, None)),     # block 0 lies behind the window of the rows from token 23 on
])
def test_rows_do_not_notice_wavefronts_whose_keys_they_do_not_see(H, d, n, window, key, blind):
    """An infinite value leaves NaN in a wavefront's sums for rows that see none of its keys (0 times infinity); these rows keep every bit."""
    cfg = I.FoldConfig("key_waves_inf", 74, 1, 4, 4, d, 64, 0, "bf16")
    assert n <= 32 or _one_unit_workgroups(4, 4, d, [16, n], window)[1]
    outs = []
    for value in (None, float("inf")):
        gpu = H.GpuFold(cfg, capacity=80, chunk_tokens=64)
        pos = 0
        for step, C in enumerate((16, n)):
            q, k, v = I.chunk_qkv(cfg, 0, step, n_tokens=C, token_base=pos)
            if value is not None and pos <= key < pos + C:
                v[key - pos, :, 5] = value
            out = gpu.step(0, q, k, v, window=window).cpu()
            pos += C
        outs.append(out)
        gpu.close()
    sees = 1 if window else key - 16  # a row of the last step that sees the key
    assert not outs[1][sees, :, 5].isfinite().any()
    differ = int((outs[0][blind] != outs[1][blind]).sum())
    assert bool(outs[0].isfinite().all()) and differ == 0
