"""Few rows that need work on their way into the cache (rotary embedding, storage round trip): the workgroups of the few-rows
kernel that read them append them themselves."""
import numpy as np
import pytest
import torch

import paper_2605_12471_amd as kv
from paper_2605_12471_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import fold_harness
    return fold_harness


# cache ends before, on and behind block and tile edges; the most rows that take this route and the first that do not (rows of a KV head
# beyond 32; with the round trip also beyond 4096 bytes of a head's keys); pieces that begin inside the chunk
@pytest.mark.parametrize("Hq,Hkv,d,chunks,splits", [
    (32, 8, 128, [130, 1, 1, 8, 9, 3], 0),
    (28, 4, 64, [63, 1, 4, 3, 5, 1, 52, 2], 0),
    (4, 4, 128, [96, 16, 17, 32, 33, 1, 31], 0),
    (4, 4, 64, [60, 32, 31, 20], 3),
    (4, 4, 128, [50, 16, 30, 9, 31], 2),
    (8, 2, 128, [64, 8, 8, 1, 15, 2], 2),
])
@pytest.mark.parametrize("rope,bits", [(True, 0), (True, 8), (True, 4), (False, 4), (False, 8)])
def test_rows_worked_on_by_their_readers_equal_the_append_kernel(H, Hq, Hkv, d, chunks, splits, rope, bits):
    """Same outputs and same cache, bit for bit, as with the append kernel in front (tuning knob)."""
    cfg = I.FoldConfig("work", 28, 1, Hq, Hkv, d, max(chunks), 0, "bf16")
    res = []
    for knob in (0, 1):
        gpu = H.GpuFold(cfg, capacity=sum(chunks), chunk_tokens=max(chunks))
        gpu.cache.set_tuning(kv.TUNE_FUSED_APPEND, knob)
        gpu.cache.set_tuning(kv.TUNE_SPLITS, splits)
        if bits:
            gpu.cache.set_storage_roundtrip(bits)
        outs, pos = [], 0
        for step, C in enumerate(chunks):
            q, k, v = I.chunk_qkv(cfg, 0, step, n_tokens=C, token_base=pos)
            gpu.cache.profile_begin(1)
            outs.append(gpu.step(0, q, k, v, **({"rope": I.rope_tables(d, pos, C)} if rope else {})).clone())
            _, append_ms, _, _ = gpu.cache.profile_end()
            takes = C * Hq // Hkv <= 32 and (not bits or C * d * 2 <= 4096)
            assert (append_ms == 0) == (knob == 0 and takes)   # the route under test is taken
            pos += C
        torch.cuda.synchronize()
        K, V = gpu.cache.view(0)
        res.append((outs, K[:, :pos].clone(), V[:, :pos].clone()))
        gpu.close()
    for a, b in zip(res[0][0], res[1][0]):
        assert torch.equal(a, b)
    assert torch.equal(res[0][1], res[1][1]) and torch.equal(res[0][2], res[1][2])


@pytest.mark.parametrize("Hq,Hkv,d,chunks,n_bits", [(32, 8, 128, [130, 1, 1, 8, 9, 3], 8), (28, 4, 64, [63, 1, 4, 3, 5, 1, 52, 2], 4)])
def test_few_rows_with_the_round_trip_under_a_window(H, oracle, Hq, Hkv, d, chunks, n_bits):
    """(The general kernel behind the append kernel.)  Output and cache against the oracle."""
    cfg = I.FoldConfig("workwin", 28, 1, Hq, Hkv, d, max(chunks), 0, "bf16")
    gpu = H.GpuFold(cfg, capacity=sum(chunks), chunk_tokens=max(chunks))
    gpu.cache.set_storage_roundtrip(n_bits)
    oc = H.make_oracle(oracle, cfg, capacity=sum(chunks))
    for step, C in enumerate(chunks):
        q, k, v = I.chunk_qkv(cfg, 0, step, n_tokens=C, token_base=oc.len)
        out = gpu.step(0, q, k, v, window=(4, 50))
        kq, vq = (oracle.storage_roundtrip(H.bits(t), n_bits) for t in (k, v))
        ref, _ = oc.step(H.wide(q), kq, vq, oc.len, n_sink=4, window=50)
        assert np.abs(H.wide(out) - ref).max() <= H.TOL["bf16"]
    H.assert_cache_bit_exact(gpu, oc)
    gpu.close()


# unsplit steps of one workgroup per head and of several, few rows, split steps (second count); other head counts: the output is longer
# than the rows and begins on them
@pytest.mark.parametrize("splits", [0, 2])
@pytest.mark.parametrize("dtype,rope,Hq,d,window", [
    ("bf16", True, 4, 64, None), ("bf16", False, 4, 64, None), ("bf16", False, 4, 128, None), ("bf16", False, 4, 128, (4, 200)),
    ("bf16", False, 8, 128, None), ("f32", False, 4, 64, None), ("f32", False, 4, 128, None),
])
def test_output_on_top_of_the_new_rows(H, dtype, rope, Hq, d, window, splits):
    """The output may take the place of k_new or v_new: the rows are used up before it is written."""
    cfg = I.FoldConfig("inplace", 29, 1, Hq, 4, d, 256, 0, dtype)
    chunks = [64, 256, 33, 1, 128, 100, 17]
    got = []
    for on in (None, "k", "v"):
        gpu = H.GpuFold(cfg, capacity=sum(chunks), chunk_tokens=256)
        gpu.cache.set_tuning(kv.TUNE_SPLITS, splits)
        outs, pos = [], 0
        for step, C in enumerate(chunks):
            q, k, v = (t.cuda().contiguous() for t in I.chunk_qkv(cfg, 0, step, n_tokens=C, token_base=pos))
            out = torch.empty_like(q)
            rows = {None: None, "k": k, "v": v}[on]
            if rows is not None:
                at = out.view(-1)[:rows.numel()].view(rows.shape)
                at.copy_(rows)
                k, v = (at, v) if on == "k" else (k, at)
            kw = {"rope": tuple(t.cuda() for t in I.rope_tables(d, pos, C))} if rope else {"window": window} if window else {}
            gpu.cache.step(0, q, k, v, out, **kw)
            outs.append(out.clone())
            pos += C
        torch.cuda.synchronize()
        K, V = gpu.cache.view(0)
        got.append(outs + [K[:, :pos].clone(), V[:, :pos].clone()])
        gpu.close()
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
