"""GPU results at the ends of the value range: infinities and NaN among the inputs, logits and
values of extreme size.  Against plain float64 arithmetic over the keys that a row sees."""
import numpy as np
import pytest
import torch

import paper_2407_20485_amd as a2sf
import parity

pytestmark = pytest.mark.gpu

CODE = {torch.float32: a2sf.A2SF_F32, torch.bfloat16: a2sf.A2SF_BF16}


def prefill(q, k, v, alpha=1.0, select=8, recent=8):
    """q [G, group, n, d]; outputs and the score of every token."""
    G, group, n, d = q.shape
    cache = a2sf.Cache(G, select + recent + 1, d, q.dtype)
    o, s = torch.full_like(q, 7.0), torch.full((G, n), 7.0, device="cuda")
    ws = torch.empty(a2sf.a2sf_workspace_bytes(G * group, n, cache.capacity, d, CODE[q.dtype], select, recent),
                     dtype=torch.uint8, device="cuda")
    a2sf.a2sf_prefill_gqa(q, k, v, n, group, alpha, select, recent, cache, o=o, scores_full=s, workspace=ws)
    torch.cuda.synchronize()
    return o, s


def chunk(q, k, v, cached, select=8, recent=8):
    """The last rows of a prompt as a chunk behind its first `cached` ones."""
    G, group, m, d = q.shape
    cache = a2sf.Cache(G, cached + m + select + recent + 1, d, q.dtype)
    cache.k[:, :cached], cache.v[:, :cached] = k[:, :cached], v[:, :cached]
    cache.scores[:, :cached] = 1.0
    cache.pos[:, :cached] = torch.arange(cached, device="cuda").int()
    cache.len.fill_(cached)
    o = torch.full_like(q, 7.0)
    ws = torch.empty(a2sf.a2sf_workspace_bytes(G * group, m, cache.capacity, d, CODE[q.dtype], select, recent),
                     dtype=torch.uint8, device="cuda")
    a2sf.a2sf_prefill_chunk_gqa(q, k[:, cached:].contiguous(), v[:, cached:].contiguous(), m, cached, group, 0.5,
                                select, recent, cache, o=o, workspace=ws)
    torch.cuda.synchronize()
    return o


def rows_by_hand(q, k, v, off=0):
    """float64 attention rows that read only the keys they see."""
    q, k, v = parity.to_f64(q), parity.to_f64(k), parity.to_f64(v)
    out = np.empty(q.shape)
    for g in range(q.shape[0]):
        for r in range(q.shape[1]):
            for i in range(q.shape[2]):
                z = k[g, : off + i + 1] @ q[g, r, i] / np.sqrt(q.shape[3])
                p = np.exp(z - z.max())
                with np.errstate(invalid="ignore"):
                    out[g, r, i] = (p / p.sum()) @ v[g, : off + i + 1]
    return out


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group,n,cached", [(1, 100, 0), (1, 200, 0), (3, 75, 0), (5, 97, 0), (1, 45, 50), (2, 33, 31)])
def test_fp32_infinities_reach_only_the_rows_that_see_them(d, group, n, cached):
    """V rows with an infinity or a NaN, each in another tile: the rows before them share the tile and
    stay finite, the rows after them get what float64 arithmetic gets."""
    gen = torch.Generator(device="cuda").manual_seed(d + n)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    q, k, v = rnd(4, group, n, d), rnd(4, cached + n, d), rnd(4, cached + n, d)
    at = cached + n - 20
    v[0, at, 3], v[1, at, d - 1], v[2, at, 7] = float("inf"), float("nan"), -float("inf")
    v[2, at + 5, 7] = float("inf")
    o = chunk(q, k, v, cached) if cached else prefill(q, k, v)[0]
    got, want = o.double().cpu().numpy(), rows_by_hand(q, k, v, cached)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.where(np.isinf(want), want, 0.0), np.where(np.isinf(got), got, 0.0))
    finite = np.isfinite(want)
    assert finite.mean() > 0.9 and np.abs(got[finite] - want[finite]).max() <= parity.O_TOL["f32"]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("size", [1e6, 1e12, 1e30, 1e34])
def test_fp32_logits_of_any_size(d, size):
    """Rows whose logits are all far below (and above) the range of an exponent: with one key, with the same
    logit for all keys, and with logits that rise or fall so steeply that one key has all the weight."""
    n = 160  # (beyond the prompts that go row by row)
    q, k = torch.zeros(6, 1, n, d, device="cuda"), torch.zeros(6, n, d, device="cuda")
    v = torch.randn(6, n, d, generator=torch.Generator(device="cuda").manual_seed(d), device="cuda")
    ramp = 1.0 + 0.01 * torch.arange(n, device="cuda")
    q[..., 0] = 1.0
    k[0, :, 0], k[1, :, 0], k[2, :, 0] = -size, -size * ramp, -size / ramp
    k[3:, :, 0] = -k[:3, :, 0]
    o = prefill(q, k, v)[0][:, 0].double()
    same = v.double().cumsum(1) / torch.arange(1, n + 1, device="cuda").view(1, n, 1)
    for g, want in ((0, same[0]), (1, v[1, :1].double()), (2, v[2].double()), (3, same[3]), (4, v[4].double()), (5, v[5, :1].double())):
        if size < 1e12 and g in (2, 5):   # the last keys' logits lie a few hundred apart, still one key's weight
            assert 1.0 / ramp[-2] - 1.0 / ramp[-1] > 100.0 * d ** 0.5 / size
        assert (o[g] - want).abs().max() <= parity.O_TOL["f32"], g


@pytest.mark.parametrize("G,n,d,cached", [(2, 200, 64, 0), (2, 200, 128, 0), (300, 200, 64, 0), (300, 200, 128, 0), (129, 1000, 128, 0),
                                          (64, 2049, 128, 0), (2, 70, 64, 130), (2, 70, 128, 130)])
def test_bf16_values_of_extreme_size(G, n, d, cached):
    """Values of 1e34 whose later keys have logits 24 octaves above the earlier ones: a row's average is a value of
    1e34 again, whatever its probabilities are taken relative to (bf16 rounds it by 2^-8 at most)."""
    total = cached + n
    q, k = torch.zeros(G, 1, n, d, device="cuda"), torch.zeros(G, total, d, device="cuda")
    q[..., 0] = 4.0
    k[:, total // 2:, 0] = 24 * np.log(2.0) * d ** 0.5 / 4
    v = torch.full((G, total, d), 1e34, device="cuda")
    v[:, ::2] *= -0.5
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    o = chunk(q, k, v, cached) if cached else prefill(q, k, v)[0]
    want = rows_by_hand(q[:1], k[:1], v[:1], cached) / 1e34
    got = o.double().cpu().numpy() / 1e34
    assert np.isfinite(got).all()
    assert np.abs(got - want).max() <= 2e-2


@pytest.mark.parametrize("L", [150, 1000, 5000, 40000])
def test_selection_among_nan_scores(L):
    """Scores that are NaN of any sign and payload, all bits set among them: every head keeps as many slots as the
    budget has, the recent ones among them, positive NaN before and negative ones after every number."""
    rng = np.random.default_rng(L)
    bits = rng.random((5, L)).astype(np.float32).view(np.uint32)
    nan = np.array([0x7FFFFFFF, 0xFFFFFFFF, 0x7FC00000, 0xFFC00000, 0xFFFFFFFE], dtype=np.uint32)
    bits[0, ::3] = rng.choice(nan, bits[0, ::3].shape)
    bits[1, :], bits[2, :], bits[3, : L // 2] = 0xFFFFFFFF, 0x7FFFFFFF, 0xFFFFFFFF
    scores = torch.from_numpy(bits.view(np.float32)).cuda()
    select, recent = L // 3, L // 7
    for pos in (None, torch.arange(L, device="cuda").int().expand(5, L).contiguous()):
        keep = torch.full((5, select + recent), -1, dtype=torch.int32, device="cuda")
        n_keep = torch.zeros(5, dtype=torch.int32, device="cuda")
        a2sf.a2sf_select(scores, pos, None, 5, L, L, select, recent, keep, n_keep)
        torch.cuda.synchronize()
        order = np.where(bits >> 31, ~bits, bits | 0x80000000).clip(1, 0xFFFFFFFE)
        order[:, L - recent:] = 0xFFFFFFFF
        for g in range(5):
            want = np.sort(np.lexsort((np.arange(L), -order[g].astype(np.int64)))[: select + recent])
            assert int(n_keep[g]) == select + recent and np.array_equal(keep[g].cpu().numpy(), want), g


@pytest.mark.parametrize("d,G,n,cached", [(64, 4, 90, 0), (64, 60, 200, 0), (64, 260, 130, 0), (128, 5, 100, 0), (128, 200, 130, 0),
                                          (64, 300, 70, 50), (128, 300, 70, 50)])
def test_fp32_infinite_operands(d, G, n, cached):
    """Infinities in K and V, finite values at the end of the range: the parts of a number whose products the matrix ops sum
    are finite for every finite number, and what an infinity does is what plain arithmetic does.  Every launch form."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    total = cached + n
    q, k, v = rnd(G, 1, n, d), rnd(G, total, d), rnd(G, total, d)
    at = total - 20
    q[0, ..., 0], k[0, at, 0] = 1.0, -float("inf")       # a key that no row gives weight
    v[1, at, 3] = 3.402823e38                            # (the largest bf16 number is smaller)
    v[2, at, 5] = -float("inf")
    k[3, at, 1] = float("nan")
    o = chunk(q, k, v, cached) if cached else prefill(q, k, v)[0]
    got = o[:4].double().cpu().numpy()
    with np.errstate(invalid="ignore"):
        want = rows_by_hand(q[:4], k[:4], v[:4], cached)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.where(np.isinf(want), want, 0.0), np.where(np.isinf(got), got, 0.0))
    finite = np.isfinite(want)
    scale = np.maximum(1.0, np.abs(np.where(finite, want, 0.0)))
    assert np.abs((np.where(finite, got, 0.0) - np.where(finite, want, 0.0)) / scale).max() <= parity.O_TOL["f32"]
    if not cached:
        s = prefill(q, k, v)[1]
        assert torch.isfinite(s[:3]).all() and s[0, at] == 0.0 and torch.isnan(s[3, at:]).any()


# fp32 prompts by tiles in every launch form (blocks per workgroup, waves), and chunks
FP32_FORMS = [(64, 21, 200, 0), (64, 60, 200, 0), (64, 260, 130, 0), (64, 300, 70, 50), (128, 11, 200, 0), (128, 200, 130, 0), (128, 300, 70, 50),
              (64, 700, 32, 0), (128, 430, 31, 0), (128, 300, 20, 50),  # one tile: one wave (the last: for the scores)
              (64, 200, 40, 0), (128, 70, 64, 0), (64, 70, 20, 13)]  # two tiles: two waves


@pytest.mark.parametrize("d,G,n,cached", FP32_FORMS)
def test_fp32_single_products(d, G, n, cached):
    """Logits that are one product each, of operands whose halves after the eighth bit are all ones (what a cut part drops is
    largest there) and of random ones: a product is off by no more than two fp32 roundings.  Seen through the probabilities:
    V is one-hot, key 0 has logit 0, all others -15 to -100."""
    rng = np.random.default_rng(d + G)
    total = cached + n
    unlucky = np.uint32(0x3F80FFFF).view(np.float32)
    mantissas = lambda shape: np.where(rng.random(shape) < 0.5, unlucky, rng.uniform(1, 2, shape)).astype(np.float32)
    q, k, v = np.zeros((G, 1, n, d), np.float32), np.zeros((G, total, d), np.float32), np.zeros((G, total, d), np.float32)
    at = rng.integers(0, d, (G, 1, n, 1))
    np.put_along_axis(q, at, mantissas(at.shape), 3)
    k[:, 1:] = -2 * d * mantissas((G, total - 1, d))
    v[:, np.arange(total), np.arange(total) % d] = 1.0
    tq, tk, tv = (torch.from_numpy(x).cuda() for x in (q, k, v))
    o, s = (chunk(tq, tk, tv, cached), None) if cached else prefill(tq, tk, tv, alpha=0.5)
    heads = sorted({0, G // 2, G - 1})
    visible = np.arange(total)[None] <= cached + np.arange(n)[:, None]
    rounding = 2.0 ** -24
    for g in heads:
        z = q[g, 0].astype(np.float64) @ k[g].astype(np.float64).T / np.sqrt(d)
        assert z[:, 1:].max() < -15 and z.min() > -100
        p = np.exp(np.where(visible, z, -np.inf))
        p /= p.sum(1, keepdims=True)
        # two roundings of the product, two of its scaling; exponential, sum and quotient: eight of the result
        off = p * rounding * (4 * np.abs(z) + 8)
        want = p @ v[g].astype(np.float64)
        seen = want > 2.0 ** -108  # (below, parts of a probability are subnormal)
        assert (np.abs(o[g, 0].double().cpu().numpy() - want) <= off @ v[g])[seen].all()
        if s is not None:
            w = 0.5 ** np.arange(n - 1, -1, -1.0)
            want = w @ p
            seen = want > 2.0 ** -108
            assert (np.abs(s[g].double().cpu().numpy() - want) <= w @ off)[seen].all()


@pytest.mark.parametrize("d,G,n,cached", [f for f in FP32_FORMS if not f[3]])
def test_fp32_products_of_one_sign_have_no_bias(d, G, n, cached):
    """Operands of one sign, a little above a power of two: an error that always has the sign of the product does not average out
    over the sum or the keys.  The mean error of the logits stays below half a rounding."""
    rng = np.random.default_rng(d + n)
    q = rng.uniform(1, 1.0078, (G, 1, n, d)).astype(np.float32)
    k = -4 * rng.uniform(1, 1.0078, (G, n, d)).astype(np.float32)
    k[:, 0] = 0
    v = rng.standard_normal((G, n, d)).astype(np.float32)
    v[..., 0] = 0
    v[:, 0] = 0
    v[:, 0, 0] = 1  # (column 0 of an output: the first key's probability)
    _, s = prefill(*(torch.from_numpy(x).cuda() for x in (q, k, v)), alpha=0.0)  # the last row's probabilities
    scale = np.float64(np.float32(np.float32(1.4426950408889634) / np.float32(np.sqrt(np.float32(d)))))
    errors = []
    for g in range(0, G, max(1, G // 20)):
        z = k[g].astype(np.float64) @ q[g, 0, -1].astype(np.float64) * scale  # (as an exponent of 2)
        got = np.log2(s[g].double().cpu().numpy())[1:]
        errors.append((got - (z - np.log2(np.exp2(z).sum()))[1:]) / z[1:])
    assert abs(np.mean(errors)) <= 2.0 ** -25, np.mean(errors) * 2 ** 24


@pytest.mark.parametrize("d,G,n,cached", FP32_FORMS)
@pytest.mark.parametrize("form", ["small q", "small k", "small v", "smallest v", "sparse v", "v of one sign"])
def test_fp32_operands_at_the_lower_end(d, G, n, cached, form):
    """Numbers whose low bf16 parts would be subnormal or nothing: results are those of fp32 arithmetic."""
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    total = cached + n
    q, k, v = rnd(G, 1, n, d), rnd(G, total, d), rnd(G, total, d)
    up = 1.0
    if form == "small q":
        q, k = q * 2.0 ** -120, k * 2.0 ** 121
    elif form == "small k":
        q, k = q * 2.0 ** 120, k * 2.0 ** -119
    elif form == "small v":
        up = 2.0 ** 112
    elif form == "smallest v":
        up = 2.0 ** 121
    elif form == "v of one sign":  # outputs of 2^-104 up: as split, low parts of which are subnormal
        up = 2.0 ** 104
        v = v.abs() + 1
    else:  # columns with one small number each among zeros, and columns of ordinary numbers
        up = 2.0 ** 110
        v[:, ::2, ::3] = 0
        v[:, 1::2, ::3] /= up
    if form in ("small v", "smallest v", "v of one sign"):
        v /= up
    o, s = (chunk(q, k, v, cached), None) if cached else prefill(q, k, v)
    heads = sorted({0, G // 2, G - 1})
    q, k, v = q[heads], k[heads], v[heads]
    want, got = rows_by_hand(q, k, v, cached), o[heads].double().cpu().numpy()
    error = np.abs(got - want)
    if form == "sparse v":
        assert error[..., ::3].max() * up <= parity.O_TOL["f32"]
        error[..., ::3] = 0
        up = 1.0
    assert error.max() * up <= parity.O_TOL["f32"]
    if form.endswith(("v", "sign")) and not cached:  # the first row has one key: its value itself, but for the order of three parts
        assert (error[:, 0, 0] <= 2.0 ** -23 * np.abs(want[:, 0, 0])).all()
    if s is not None:
        mask = np.tril(np.ones((n, n), bool))
        for i, g in enumerate(heads):
            z = parity.to_f64(q[i, 0]) @ parity.to_f64(k[i]).T / np.sqrt(d)
            p = np.exp(np.where(mask, z, -np.inf))
            want = (p / p.sum(1, keepdims=True)).sum(0)
            assert (np.abs(s[g].double().cpu().numpy() - want) / want).max() <= parity.SCORE_RTOL


@pytest.mark.parametrize("d,G,n,cached", [f for f in FP32_FORMS if not f[3]])
def test_fp32_large_logits_beside_infinities(d, G, n, cached):
    """Logits of 1e7 and more, whose last bits decide: an infinity in V changes neither the scores nor any other output, and one in a key
    that gets no weight either way changes nothing at all."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    q, k, v = rnd(G, 1, n, d) * 3e3, rnd(G, n, d) * 3e3, rnd(G, n, d)
    q[..., 0] = 1.0
    at = n - 20
    k[:, at] = 0
    k[:, at, 0] = -1e30
    o, s = prefill(q, k, v)
    assert torch.isfinite(s).all() and torch.isfinite(o).all()
    v[:, 3, 5], v[:, n // 2, 7] = float("inf"), float("nan")
    o2, s2 = prefill(q, k, v)
    assert torch.equal(s, s2)
    same = torch.ones_like(o, dtype=torch.bool)
    same[:, :, 3:, 5], same[:, :, n // 2:, 7] = False, False
    assert torch.equal(o[same], o2[same])
    assert not torch.isfinite(o2[:, :, 3:, 5]).any() and torch.isnan(o2[:, :, n // 2:, 7]).all()
    v[:, 3, 5], v[:, n // 2, 7] = 0.25, 0.25
    o, s = prefill(q, k, v)
    k[:, at, 0] = -float("inf")
    o2, s2 = prefill(q, k, v)
    assert torch.equal(s, s2) and torch.equal(o, o2)
