"""KvFoldCache.step: its native form takes what the plain Python one takes, with the same results, and leaves the rest to it."""
import importlib.util
import threading

import pytest
import torch

import paper_2605_12471_amd as kv
from paper_2605_12471_amd import binding, build
from paper_2605_12471_amd import inputs as I

N, HQ, HKV, D = 24, 8, 2, 64


def test_the_native_step_is_built_for_this_torch():
    assert binding._native_step() is not None


@pytest.mark.parametrize("fails", ["no source", "no compiler"])
def test_a_build_without_it_goes_on(monkeypatch, tmp_path, capfd, fails):
    """Where the native step does not compile the build leaves none, also not an older one, and the plain Python step serves."""
    path = tmp_path / "kvfold_py_step.so"
    path.write_bytes(b"of an earlier build")
    monkeypatch.setattr(build, "PY_STEP_PATH", str(path))
    if fails == "no compiler":
        monkeypatch.setenv("PATH", str(tmp_path))
    else:
        monkeypatch.setattr(build, "CSRC", str(tmp_path))   # (there is no py_step.cpp)
    assert build.build_py_step() is None and not path.exists()
    assert "native step" in capfd.readouterr().err


def test_two_threads_whose_first_steps_meet_both_have_it(monkeypatch):
    """A thread that looks for the native step while another one is loading it does not take it for missing."""
    monkeypatch.setattr(binding, "_native", False)
    loading, go_on, real, got = threading.Event(), threading.Event(), importlib.util.module_from_spec, {}

    def slow(spec):
        loading.set()
        assert go_on.wait(10)
        return real(spec)
    monkeypatch.setattr(importlib.util, "module_from_spec", slow)
    first, second = (threading.Thread(target=lambda i=i: got.__setitem__(i, binding._native_step())) for i in (0, 1))
    first.start()
    assert loading.wait(10)
    second.start()
    second.join(0.2)   # (looked already, or waits)
    go_on.set()
    first.join(10)
    second.join(10)
    assert got[0] is not None and got[1] is got[0]


@pytest.fixture()
def cache():
    c = kv.KvFoldCache(2, HQ, HKV, D, 64, 256, "bf16")
    yield c
    c.close()


def _args(seed=1, n=N):
    g = torch.Generator("cuda").manual_seed(seed)
    q, k, v = (torch.randn(n, h, D, generator=g, device="cuda").bfloat16() for h in (HQ, HKV, HKV))
    return q, k, v, torch.zeros_like(q)


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["plain", "lse", "noalloc", "rope", "window", "stream"])
def test_the_same_step_either_way(cache, form):
    kw = {"noalloc": {"noalloc": True}, "window": {"window": (2, 9)}, "rope": {"rope": I.rope_tables(D, 0, N, device="cuda")},
          "lse": {"lse": torch.zeros(HQ, N, device="cuda")}, "stream": {"stream": torch.cuda.current_stream().cuda_stream}}.get(form, {})
    q, k, v, out = _args()
    got = []
    for native in (True, False):
        cache._bound = False if native else None
        cache.set_length(-1, 0)
        out.zero_()
        assert cache.step(1, q, k, v, out, **kw) is out
        assert (cache._bound is not None) == native
        got.append([out.clone()] + [t[:, :N].clone() for t in cache.view(1)] + ([kw["lse"].clone()] if form == "lse" else []))
        assert cache.length(1) == N and cache.length(0) == 0
    assert all(torch.equal(a, b) for a, b in zip(*got)) and got[0][0].any()


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_what_is_refused(cache, native):
    cache._bound = False if native else None
    q, k, v, out = _args()
    tables = I.rope_tables(D, 0, N, device="cuda")
    refused = [
        (ValueError, (q.float(), k, v, out), {}), (ValueError, (q, k.cpu(), v, out), {}), (ValueError, (q, k, v[:, :1], out), {}),
        (ValueError, (q, k, v, out.transpose(0, 1)), {}), (ValueError, (q[0], k, v, out), {}),
        (ValueError, (q, k, v, out), {"lse": torch.zeros(N, HQ, device="cuda")}), (ValueError, (q, k, v, out), {"rope": tables, "noalloc": True}),
        (ValueError, (q, k, v, out), {"rope": (tables[0], tables[1][1:])}), (AttributeError, (q, k, v, None), {}),
        (kv.KvFoldError, (q, k, v, out), {"pos_offset": 3}), (kv.KvFoldError, (q, k, v, out), {"window": (-1, 5)}),
        (kv.KvFoldError, tuple(t[:0] for t in (q, k, v, out)), {}),
    ]
    for error, args, kw in refused:
        with pytest.raises(error):
            cache.step(0, *args, **kw)
    with pytest.raises(kv.KvFoldError):
        cache.step(2, q, k, v, out, pos_offset=0)
    assert cache.length(0) == 0 and not out.any()
    cache.step(0, q, k, v, out)
    assert cache.length(0) == N


@pytest.mark.gpu
def test_after_close():
    c = kv.KvFoldCache(1, HQ, HKV, D, 64, 256, "bf16")
    q, k, v, out = _args()
    c.step(0, q, k, v, out)
    c.close()
    with pytest.raises(kv.KvFoldError):
        c.step(0, q, k, v, out, pos_offset=N)


@pytest.mark.gpu
def test_the_current_stream_is_the_callers(cache):
    """Work of another stream that the step has to wait for: on that stream it does."""
    q, k, v, out = _args()
    cache.step(0, q, k, v, out)
    torch.cuda.synchronize()
    want = out.clone()
    side, late = torch.cuda.Stream(), torch.zeros_like(q)
    cache.set_length(0, 0)
    with torch.cuda.stream(side):
        big = torch.randn(4096, 4096, device="cuda")
        for _ in range(8):
            big = big @ big * 1e-2
        late.copy_(q)
        cache.step(0, late, k, v, out)
    side.synchronize()
    assert torch.equal(out, want)
