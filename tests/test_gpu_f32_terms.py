"""fp32 mode on operands split into three bf16 terms: both workgroup sizes around the edges of the 32-key tile, values over
many powers of two, and rows that are not finite (which take the fp32 instructions)."""
import math

import pytest
import torch

import paper_2605_12471_amd as kv
from paper_2605_12471_amd import inputs as I
from test_gpu_parity_small import H, _run_case  # noqa: F401  (H: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("waves", [1, 2])  # four or eight wavefronts
@pytest.mark.parametrize("chunks", [[1, 31, 1, 31], [33, 63, 32, 65], [300, 17, 64]])
@pytest.mark.parametrize("splits", [1, 3])
def test_tile_edges(H, oracle, d, waves, chunks, splits):
    cfg = I.FoldConfig("f32_edges", 63, 1, 6, 2, d, max(chunks), 0, "f32")
    _run_case(H, oracle, cfg, chunks, splits=splits, upw=waves)


def _step(q, k, v, waves, splits, want_lse=False):
    n, hq, d = q.shape
    hkv = k.shape[1]
    cache = kv.KvFoldCache(1, hq, hkv, d, n, n, "f32")
    cache.set_tuning(0, splits)
    cache.set_tuning(1, waves)
    out = torch.empty_like(q)
    lse = torch.empty((hq, n), device="cuda") if want_lse else None
    cache.step(0, q, k, v, out, pos_offset=0, lse=lse)
    torch.cuda.synchronize()
    cache.close()
    return (out, lse) if want_lse else out


def _reference(q, k, v):
    n, hq, d = q.shape
    g = hq // k.shape[1]
    qd = q.cpu().double().transpose(0, 1)
    kd, vd = (t.cpu().double().repeat_interleave(g, dim=1).transpose(0, 1) for t in (k, v))
    s = qd @ kd.transpose(1, 2) / math.sqrt(d)
    s = s.masked_fill(torch.ones(n, n).triu(1).bool(), -math.inf)
    return (torch.softmax(s, -1) @ vd).transpose(0, 1)


def _random(n, h, d, seed):
    return torch.randn(n, h, d, generator=torch.Generator("cuda").manual_seed(seed), device="cuda")


@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("d", [64, 128])
def test_values_over_many_powers_of_two(d, waves):
    """Columns scaled by 2^-40 ... 2^40 (queries the other way round, so that the logits stay of ordinary size).  Every
    operand keeps its 24 bits; each product and sum has the fp32 bound d 2^-24 of its terms, here twice that for the two
    products, on logits below 8 (weights move by as much as their logits), and relative to the column's largest value."""
    n, hq, hkv = 200, 4, 1
    scale = 2.0 ** torch.linspace(-40, 40, d, device="cuda").round()
    q, k, v = _random(n, hq, d, 1) / scale, _random(n, hkv, d, 2) * scale, _random(n, hkv, d, 3) * scale
    out = _step(q, k, v, waves, 1)
    err = (out.cpu().double() - _reference(q, k, v)).abs() / scale.cpu().double() / 4.0
    assert err.max() <= 2 * 8 * d * 2.0 ** -24


@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("d", [64, 128])
def test_values_that_are_not_finite(d, waves, splits):
    """An infinite value, a key that hides itself (logit -inf), a key that wins alone (+inf: NaN), a NaN query."""
    n, hq, hkv = 150, 4, 2
    q, k, v = _random(n, hq, d, 4), _random(n, hkv, d, 5), _random(n, hkv, d, 6)
    q[:, :2, 3] = -q[:, :2, 3].abs()  # KV head 0: every query sees key 20 at -inf
    k[20, 0, 3] = math.inf
    v[0, 1, 7] = math.inf             # KV head 1: a value that every row sees
    q[99, 1] = math.nan
    out, ref = _step(q, k, v, waves, splits).cpu().double(), _reference(q, k, v)
    finite = torch.isfinite(ref)
    assert torch.isnan(out[99, 1]).all() and (out[:, 2:, 7] == math.inf).all()
    finite[99, 1] = False
    assert torch.equal(torch.isfinite(out), finite)
    assert (out - ref)[finite].abs().max() <= 1e-5
    # a query of the other sign sees the same key at +inf: NaN from there on, as inf - inf
    q[140, 0, 3] = 1.0
    out = _step(q, k, v, waves, splits).cpu()
    assert torch.isnan(out[140, 0]).all() and torch.isfinite(out[139, 0]).all()


@pytest.mark.parametrize("d", [64, 128])
def test_largest_finite_values(d):
    """The largest floats are split without overflow (the leading term is rounded towards zero)."""
    n, big = 40, 3.4028234663852886e38
    q = torch.zeros(n, 1, d, device="cuda")
    k, v = _random(n, 1, d, 7), torch.zeros(n, 1, d, device="cuda")
    v[0, 0, 5] = big
    out = _step(q, k, v, 1, 1).cpu().double()[:, 0, 5]
    ref = big / torch.arange(1, n + 1, dtype=torch.float64)
    assert ((out - ref).abs() <= 8 * 2.0 ** -24 * ref).all()


@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("d", [64, 128])
def test_finite_values_whose_product_overflows(d, waves):
    """Key 20 is -FLT_MAX in one column and the queries 2^24 there: its logit is -infinity in 32 bits, its weight 0, and
    every row keeps the finite result of the other keys (an error of the other logits is one of 128 products: 1e-5)."""
    n, hq, hkv = 70, 4, 2
    q, k, v = _random(n, hq, d, 8), _random(n, hkv, d, 9), _random(n, hkv, d, 10)
    k[:, :, 3] = 0.0
    k[20, :, 3] = -3.4028234663852886e38
    q[:, :, 3] = 2.0 ** 24
    out, ref = _step(q, k, v, waves, 1).cpu().double(), _reference(q, k, v)
    assert torch.isfinite(out).all()
    assert (out - ref).abs().max() <= 1e-5


@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("d", [64, 128])
def test_smallest_values_keep_their_bits(d, waves):
    """Values of 2^-120 come out as the same values of ordinary size do, 2^-120 smaller: both are sums of the same numbers,
    which differ by roundings of 2^-24 of the largest (here allowed sixteen).  A third term below the smallest bf16 number
    would leave 2^-14 of a value."""
    n, hq, hkv = 100, 4, 2
    q, k = _random(n, hq, d, 11), _random(n, hkv, d, 12)
    v = _random(n, hkv, d, 13)
    v = torch.copysign(1.0 + torch.frac(v.abs()), v)
    small, plain = (_step(q, k, v * s, waves, 1).cpu().double() / s for s in (2.0 ** -120, 1.0))
    assert (small - plain).abs().max() <= 2.0 ** -20


@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("d", [64, 128])
def test_single_products_are_rounded_once(d, waves):
    """Row i's query has one column, which only key i has too: its log-sum-exp is one product.  The six roundings on the way
    (product, scale, its constant, reference + log, ln 2, its constant) are each at most 2^-24 and on average nothing, where
    products of second and third terms would be missing by 4 x 2^-24 of the product, all of one sign for these numbers:
    the lower 16 bits of a factor are 2^-7 - 2^-16 - something, as second and third term 2^-7 - 2^-15 and 2^-16 - something."""
    n, h = 64, 8
    gen = torch.Generator().manual_seed(14)
    def factor():
        return 1.0 + torch.randint(0, 16, (n, h), generator=gen) / 128 + 2.0 ** -7 - 2.0 ** -16 - torch.randint(0, 16, (n, h), generator=gen) * 2.0 ** -23
    x, y = factor() * 512.0, factor()
    q, k = torch.zeros(n, h, d), torch.zeros(n, h, d)
    i = torch.arange(n)
    q[i, :, i], k[i, :, i] = x, y
    lse = _step(q.cuda(), k.cuda(), _random(n, h, d, 15), waves, 1, want_lse=True)[1].cpu().double().T
    exact = x.double() * y.double() / math.sqrt(d)
    err = lse / exact - 1.0
    assert err.abs().max() <= 6 * 2.0 ** -24
    assert err.mean().abs() <= 2.0 ** -24


@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("d", [64, 128])
def test_rows_do_not_notice_what_they_do_not_see(d, waves, splits):
    """A key that is not finite changes no bit of the rows before it, wherever they are computed, and a query that is not
    finite changes no bit of any other row."""
    n, hq, hkv = 200, 4, 2
    q, k, v = _random(n, hq, d, 16), _random(n, hkv, d, 17), _random(n, hkv, d, 18)
    plain = _step(q, k, v, waves, splits)
    k2, v2, q2 = k.clone(), v.clone(), q.clone()
    k2[150, 0, 3] = math.nan
    v2[160, 1, 7] = math.inf
    out = _step(q, k2, v2, waves, splits)
    assert torch.equal(out[:150, :2], plain[:150, :2]) and torch.isnan(out[150:, :2]).all()
    assert torch.equal(out[:160, 2:], plain[:160, 2:]) and (out[160:, 2:, 7] == math.inf).all()
    ref = _reference(q, k2, v2)[160:, 2:]
    assert (out[160:, 2:].cpu().double() - ref)[torch.isfinite(ref)].abs().max() <= 1e-5
    q2[77, 1, 5] = math.nan
    out = _step(q2, k, v, waves, splits)
    assert torch.isnan(out[77, 1]).all()
    out[77, 1] = plain[77, 1]
    assert torch.equal(out, plain)


@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("waves", [1, 2])
def test_many_keys_that_are_not_finite(waves, splits):
    """Every tile of 32 keys, more of them than a workgroup takes one by one, holds a value or a key that is not finite: the
    column with infinite values is not finite from the first such key on, hidden keys (-inf) have no weight, all else is as ever."""
    n, hq, hkv, d = 1500, 2, 1, 64
    q, k, v = _random(n, hq, d, 19), _random(n, hkv, d, 20), _random(n, hkv, d, 21)
    q[:, :, 3] = -q[:, :, 3].abs() - 0.1
    k[5::37, 0, 3] = math.inf
    v[7::29, 0, 9] = math.inf
    out, ref = _step(q, k, v, waves, splits).cpu().double(), _reference(q, k, v)
    cols = torch.arange(d) != 9
    assert (out[..., cols] - ref[..., cols]).abs().max() <= 1e-5
    assert not torch.isfinite(out[7:, :, 9]).any()


@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("d", [64, 128])
def test_values_and_queries_beyond_the_terms_with_the_rotary_embedding(H, oracle, d, waves):
    """The fp32 instructions rotate the queries that they take from memory: the same bits as on inputs rotated beforehand."""
    cfg = I.FoldConfig("f32_rope", 71, 1, 4, 2, d, 100, 0, "f32")
    q, k, v = I.chunk_qkv(cfg, 0, 0)
    v[10, 0, 5] = 2.0 ** 70
    q[60, 1, 3] = 2.0 ** 61
    k[:, :, [3, 3 + d // 2]] *= 2.0 ** -60  # (a pair of the rotation: logits of ordinary size)
    cos, sin = I.rope_tables(d, 0, 100)
    q_rot, k_rot = (torch.from_numpy(oracle.rope(t.numpy(), cos.numpy(), sin.numpy())) for t in (q, k))
    outs = []
    for args, rope in (((q, k, v), (cos, sin)), ((q_rot, k_rot, v), None)):
        fold = H.GpuFold(cfg, capacity=100)
        fold.cache.set_tuning(1, waves)
        outs.append(fold.step(0, *args, rope=rope).cpu())
        fold.close()
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(*outs)


@pytest.mark.parametrize("splits", [0, 2])
@pytest.mark.parametrize("waves", [1, 2])
@pytest.mark.parametrize("d", [64, 128])
def test_values_beyond_the_terms_under_a_window(H, oracle, d, waves, splits):
    """Key 150 holds a value of 2^65 and a window of 40 keys passes over it: the rows that see it match the oracle (relative to
    that value), all others keep every bit."""
    n, window = 300, (2, 40)
    cfg = I.FoldConfig("f32_window", 72, 1, 4, 2, d, n, 0, "f32")
    q, k, v = I.chunk_qkv(cfg, 0, 0)
    big = v.clone()
    big[150, :, 9] = 2.0 ** 65
    outs = []
    for value in (v, big):
        fold = H.GpuFold(cfg, capacity=n)
        fold.cache.set_tuning(0, splits)
        fold.cache.set_tuning(1, waves)
        outs.append(fold.step(0, q, k, value, window=window).cpu())
        fold.close()
    sees = torch.zeros(n, dtype=torch.bool)
    sees[150:150 + window[1]] = True
    assert torch.equal(outs[0][~sees], outs[1][~sees])
    ref = torch.from_numpy(H.oracle_step(H.make_oracle(oracle, cfg, capacity=n), q, k, big, window=window)[0])
    err = (outs[1].double() - ref).abs()
    cols = torch.arange(d) != 9
    assert err[..., cols].max() <= 1e-5
    assert (err[sees][..., 9] <= 1e-5 * ref[sees][..., 9].abs()).all()
