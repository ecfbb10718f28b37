"""fp32: the attention kernel appends the chunk's rows itself and reads them as handed in."""
import pytest
import torch

import paper_2605_12471_amd as kv
from paper_2605_12471_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    from tests import fold_harness
    return fold_harness


# (The kernel has a form of four wavefronts and one of eight; the first appends, in pieces of fewer than 20 tiles, 12 where heads are
# 64 wide.  waves = 4 asks for it whatever the plan says.)
@pytest.mark.parametrize("Hq,Hkv,d,chunks,splits,window,odd,waves,appends", [
    (4, 1, 64, [128] * 4, 0, None, None, 0, None),                  # the short fold: a few tiles per step
    (8, 2, 128, [1, 31, 32, 33, 63, 64, 65, 1], 0, None, None, 4, None),   # the cache's end before, on and behind every edge of a half tile
    (28, 4, 128, [300, 7, 500], 3, None, None, 4, None),            # pieces that end before the chunk begins, inside it, and behind it
    (28, 4, 128, [70, 100, 130], 5, None, None, 4, None),
    (6, 6, 64, [200, 1, 90], 2, (4, 100), None, 4, None),           # sinks and window, some of them in the chunk
    (6, 2, 128, [100, 300, 33], 3, (100, 60), None, 4, None),
    (4, 4, 128, [100, 60], 0, None, (0, 150), 4, None),             # a key of the old cache and one of the chunk for the fp32 instructions
    (4, 4, 64, [60, 100], 2, None, (59, 60, 130), 4, None),
    (4, 2, 128, [1100, 116, 64, 9], 1, None, (1099, 1270), 4, [True, True, False, False]),  # 18, 19, 20 and 21 tiles a piece
    (4, 2, 64, [600, 104, 64, 9], 1, None, (599, 750), 4, [True, True, False, False]),      # 10, 11, 12 and 13
])
def test_append_in_the_fp32_kernel_equals_separate_append(H, Hq, Hkv, d, chunks, splits, window, odd, waves, appends):
    """Same outputs and same cache, bit for bit, as with the append kernel in front (tuning knob)."""
    cfg = I.FoldConfig("f32append", 27, 1, Hq, Hkv, d, max(chunks), 0, "f32")
    res = []
    for knob in (0, 1):
        gpu = H.GpuFold(cfg, capacity=sum(chunks), chunk_tokens=max(chunks))
        gpu.cache.set_tuning(kv.TUNE_FUSED_APPEND, knob)
        gpu.cache.set_tuning(kv.TUNE_SPLITS, splits)
        gpu.cache.set_tuning(kv.TUNE_UNITS_PER_WAVE, waves // 4)
        outs, pos = [], 0
        for step, C in enumerate(chunks):
            q, k, v = I.chunk_qkv(cfg, 0, step, n_tokens=C, token_base=pos)
            for at in odd or ():
                if pos <= at < pos + C:
                    v[at - pos, 0, 3] = 2.0 ** 100
            kw = {} if window is None else {"window": window}
            gpu.cache.profile_begin(1)
            outs.append(gpu.step(0, q, k, v, **kw).clone())
            _, append_ms, _, _ = gpu.cache.profile_end()
            assert (append_ms == 0) == (knob == 0 and (appends is None or appends[step]))   # the route under test is taken
            pos += C
        torch.cuda.synchronize()
        K, V = gpu.cache.view(0)
        res.append((outs, K[:, :pos].clone(), V[:, :pos].clone()))
        gpu.close()
    for a, b in zip(res[0][0], res[1][0]):
        assert torch.equal(a, b)
    assert torch.equal(res[0][1], res[1][1]) and torch.equal(res[0][2], res[1][2])
