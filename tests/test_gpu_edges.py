"""GPU parity of the kernels at the edges of their tiles: remainders, the
smallest sizes of each variant and the sizes on either side of a dispatch line."""

import numpy as np
import pytest
import torch

from paper_2605_06892_amd import hsa_step as H

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _gen(seed):
    return torch.Generator(device="cpu").manual_seed(seed)


def _attend64(q, k, v, heads):
    n, d = q.shape
    dh = d // heads
    o = torch.empty(n, d, dtype=torch.float64)
    for h in range(heads):
        c = slice(h * dh, (h + 1) * dh)
        s = torch.softmax(q[:, c].double() @ k[:, c].double().t() * dh ** -0.5, dim=1)
        o[:, c] = s @ v[:, c].double()
    return o


# queries around the 16- and 32-query workgroups, rows around the 32-key blocks and the 8 waves'
# share of 256; the launches of 16 heads take 32-query workgroups on 256 compute units, the others 16
@pytest.mark.parametrize("n_q,n_kv,heads,dh", [
    (1, 1, 1, 64), (15, 31, 2, 64), (16, 32, 1, 128), (17, 33, 2, 128), (31, 255, 3, 64), (33, 257, 2, 64),
    (33, 289, 2, 128), (300, 77, 16, 64), (300, 290, 16, 128), (289, 512, 16, 64),
])
@pytest.mark.parametrize("spread", [1.0, 30.0])
def test_attention_f32_edges(n_q, n_kv, heads, dh, spread):
    """spread 30: scores hundreds apart, so most probabilities underflow."""
    g = _gen(n_q * 1000 + n_kv)
    d = heads * dh
    q, k, v = (torch.randn(n, d, generator=g) for n in (n_q, n_kv, n_kv))
    q *= spread
    out = torch.full((n_q + 1, d), 7.0, device=DEV)
    H.hsa_attention_core(q.to(DEV), k.to(DEV), v.to(DEV), n_q, heads, dh, dh ** -0.5, out)
    want = _attend64(q, k, v, heads)
    # a score of magnitude s carries an error of about dh/2 ulps of s / sqrt(dh) at most, which is
    # the relative error of its probability; the sums add a few ulps
    bar = 2.0 ** -24 * (64 + 8 * spread * dh ** 0.5)
    assert float((out[:n_q].cpu().double() - want).abs().max() / want.abs().max()) < bar
    assert torch.all(out[n_q] == 7.0)


def test_attention_f32_infinite_and_nan_scores():
    """A -inf score has probability 0, a NaN score makes its own row NaN and no other."""
    g = _gen(5)
    q, k, v = torch.rand(3, 64, generator=g) + 0.5, torch.randn(300, 64, generator=g), torch.randn(300, 64, generator=g)
    k[40:100] = -float("inf")  # whole blocks of one wave's share among them
    q[1, 3] = float("nan")
    out = torch.empty(3, 64, device=DEV)
    H.hsa_attention_core(q.to(DEV), k.to(DEV), v.to(DEV), 3, 1, 64, 0.125, out)
    keep = torch.cat([torch.arange(40), torch.arange(100, 300)])
    want = _attend64(q[[0, 2]], k[keep], v[keep], 1)
    got = out.cpu()
    assert float((got[[0, 2]].double() - want).abs().max()) < 1e-5
    assert torch.isnan(got[1]).all()


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("n_kv", [1, 33, 256, 300])
def test_attention_f32_infinite_value_in_the_last_row(n_kv, dh):
    """Rows past n_kv take no part, so an infinite value of the last row stays itself. The scores are equal: every
    row has weight."""
    g = _gen(n_kv)
    q, k, v = torch.randn(20, dh, generator=g), torch.ones(n_kv, dh), torch.randn(n_kv, dh, generator=g)
    v[-1, 3], v[-1, 5] = float("inf"), -float("inf")
    out = torch.empty(20, dh, device=DEV)
    H.hsa_attention_core(q.to(DEV), k.to(DEV), v.to(DEV), 20, 1, dh, dh ** -0.5, out)
    want = v.double().mean(0)
    got = out.cpu().double()
    assert bool((got[:, 3] == float("inf")).all()) and bool((got[:, 5] == -float("inf")).all())
    finite = want.isfinite()
    # equal weights: n_kv additions of values of size 1, each a few ulps off at most
    assert float((got[:, finite] - want[finite]).abs().max()) < 2.0 ** -24 * (16 + n_kv)


# 16 and, with 16 heads, 32 queries a workgroup
@pytest.mark.parametrize("n_q,heads,dh", [(20, 2, 64), (20, 2, 128), (300, 16, 64), (300, 16, 128)])
def test_attention_f32_four_byte_alignment(n_q, heads, dh):
    """fp32 arrays need no more than 4-byte alignment: arrays that start one float into a row give the same bits."""
    g = _gen(n_q + dh)
    d, n_kv = heads * dh, 77
    q, k, v = (torch.randn(n, d, generator=g).to(DEV) for n in (n_q, n_kv, n_kv))
    want = torch.empty(n_q, d, device=DEV)
    H.hsa_attention_core(q, k, v, n_q, heads, dh, dh ** -0.5, want)
    shifted = [torch.empty(t.numel() + 1, device=DEV)[1:].view(t.shape) for t in (q, k, v)]
    for a, b in zip(shifted, (q, k, v)):
        a.copy_(b)
    whole = torch.full((n_q * d + 2,), 7.0, device=DEV)
    out = whole[1:-1].view(n_q, d)
    H.hsa_attention_core(*shifted, n_q, heads, dh, dh ** -0.5, out)
    assert torch.equal(out, want)
    assert float(whole[0]) == 7.0 and float(whole[-1]) == 7.0


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("size", [1e2, 1e4, 3e4, 1e6])
def test_attention_f32_large_scores(size, dh):
    """Scores up to 1e13: every row's softmax is its largest score alone, as the gaps between them are."""
    g = _gen(int(size))
    q, k, v = (torch.randn(n, dh, generator=g) for n in (20, 300, 300))
    q, k = q * size, k * size
    want = _attend64(q, k, v, 1)
    out = torch.empty(20, dh, device=DEV)
    H.hsa_attention_core(q.to(DEV), k.to(DEV), v.to(DEV), 20, 1, dh, dh ** -0.5, out)
    # weights 1 and 0: a sum, a merge and a division of one value
    assert float((out.cpu().double() - want).abs().max()) < 2.0 ** -22 * float(v.abs().max())


# rows and columns around the 32 and 64 tiles, k around the 4-float loads and the slabs; 300 x 96 x 3
# outputs take the split-k tiles, 1500 x 1100 the 64 x 64 tiles on 256 compute units
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (31, 33, 3), (33, 31, 63), (65, 64, 64), (300, 96, 65), (1500, 1100, 37),
                                   (1537, 1025, 96)])
@pytest.mark.parametrize("option", ["plain", "scale_gelu", "residual"])
def test_linear_f32_edges(m, n, k, option):
    g = _gen(m + n + k)
    x, w, r = torch.randn(m, k, generator=g), torch.randn(n, k, generator=g), torch.randn(m, n, generator=g)
    s = torch.rand(m, generator=g) + 0.5
    y = torch.full((m + 1, n), 7.0, device=DEV)
    want = x.double() @ w.double().t()
    kw = {}
    if option == "scale_gelu":
        kw = {"row_scale": s.to(DEV), "gelu": True}
        z = want * s.double()[:, None]
        want = 0.5 * z * (1 + torch.tanh(np.sqrt(2 / np.pi) * (z + 0.044715 * z ** 3)))
    elif option == "residual":
        kw = {"residual": r.to(DEV)}
        want = want + r.double()
    H.hsa_linear(x.to(DEV), m, w.to(DEV), y, **kw)
    # k sums of products of size sqrt(k) ulps each, a few ulps for the epilogue
    bar = 2.0 ** -24 * (16 + 4 * k ** 0.5) * max(1.0, float(want.abs().max()))
    assert float((y[:m].cpu().double() - want).abs().max()) < bar
    assert torch.all(y[m] == 7.0)


def _ranked_budgets(keys, groups):
    """Budgets from the ascending order of (bit pattern, token), NaNs as one canonical NaN."""
    keys = np.where(np.isnan(keys), np.float64("nan"), keys)
    bits = keys.view(np.uint64)
    budget = np.empty(len(keys), np.int32)
    order = np.lexsort((np.arange(len(keys)), bits))
    at = 0
    for s, c in groups:
        budget[order[at:at + c]] = s
        at += c
    return budget


def _keys(pattern, n, rng):
    k = rng.chisquare(64, n)
    if pattern == "equal":
        return np.full(n, 2.5)
    if pattern == "two_values":
        return np.where(rng.random(n) < 0.5, 1.0, 3.0)
    if pattern == "outliers":  # the range spans every exponent, nearly all keys share a few bins
        k[rng.integers(0, n, 3)] = (0.0, np.inf, np.nan)
        return 1.0 + k * 1e-12
    if pattern == "many_nan":
        k[rng.random(n) < 0.6] = np.nan
        return k
    if pattern == "negative":
        return k - 64
    if pattern == "lognormal":
        return np.exp(4 * rng.standard_normal(n))
    if pattern == "levels":  # most boundaries among equal keys, each level a bin of its own
        return rng.integers(1, 17, n).astype(np.float64)
    if pattern == "levels_and_outlier":  # several levels share a bin, and each boundary a level with others
        k = 1.0 + rng.integers(0, 6, n) * 2.0 ** -40
        k[rng.integers(0, n)] = 1e300
        return k
    if pattern == "descending":  # within the bin of an outlier, so every key is a new minimum of it
        k = 1.0 + 1e-9 * np.arange(n, 0, -1)
        k[0] = 1e300
        return k
    return k


# tokens around a wave, the workgroup, the list, the last of the all-pairs kernel (5120) and of the selection
# with 8, 32 and 80 keys a thread in registers (8192, 32768, 81920), and beyond, where they are read again
@pytest.mark.parametrize("n", [1, 2, 17, 63, 1025, 4097, 5120, 5121, 8192, 8193, 32768, 32769, 75601, 81920, 81921,
                               100003])
@pytest.mark.parametrize("pattern", ["chi2", "equal", "two_values", "outliers", "many_nan", "negative", "lognormal",
                                     "levels", "levels_and_outlier", "descending"])
@pytest.mark.parametrize("n_groups", [1, 3, 16])
def test_assign_budgets_by_key_edges(n, pattern, n_groups):
    rng = np.random.default_rng(n * 31 + n_groups)
    T = 2 ** 15
    budgets = [2 ** i for i in range(n_groups)]
    cuts = np.sort(rng.integers(0, n + 1, n_groups - 1))
    if n_groups > 4:
        cuts[3] = cuts[2]  # an empty group
        cuts[0] = 0        # and an empty first group
    sizes = np.diff(np.concatenate([[0], cuts, [n]]))
    groups = list(zip(budgets, sizes.tolist()))
    keys = _keys(pattern, n, rng)
    out = torch.full((n + 1,), -5, dtype=torch.int32, device=DEV)
    H.hsa_assign_budgets_by_key(torch.from_numpy(keys).to(DEV), T, groups, out[:n])
    assert np.array_equal(out[:n].cpu().numpy(), _ranked_budgets(keys, groups))
    assert int(out[n]) == -5


@pytest.mark.parametrize("n", [5121, 8193, 32769, 81919])
def test_assign_budgets_by_key_at_the_end_of_an_allocation(n):
    """The keys are the last bytes of a 32 MiB device allocation, a segment of its own: a read past them leaves it."""
    rng = np.random.default_rng(n)
    keys = rng.chisquare(64, n)
    whole = torch.empty((32 << 20) // 8, dtype=torch.float64, device=DEV)
    whole[-n:] = torch.from_numpy(keys)
    groups = [(1, n // 3), (2, n // 3), (4, n - 2 * (n // 3))]
    out = torch.empty(n, dtype=torch.int32, device=DEV)
    H.hsa_assign_budgets_by_key(whole[-n:], 4, groups, out)
    assert np.array_equal(out.cpu().numpy(), _ranked_budgets(keys, groups))


# tokens around the 32 of a workgroup, channels around the 64 of a chunk and off the 16-byte path
@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 1000])
@pytest.mark.parametrize("channels", [4, 16, 62, 64, 68, 200])
def test_l1_rel_edges(n, channels):
    rng = np.random.default_rng(n + channels)
    v, p = (rng.standard_normal((n, channels)).astype(np.float32) for _ in range(2))
    v[0] = 0.0  # x/0
    acc0 = rng.random(n)
    num, den = np.zeros(n), np.zeros(n)
    for c in range(channels):  # float64 sums in channel order
        num += np.abs(v[:, c].astype(np.float64) - p[:, c].astype(np.float64))
        den += np.abs(v[:, c].astype(np.float64))
    with np.errstate(divide="ignore"):
        want = acc0 + num / den
    tv, tp, ta = (torch.from_numpy(a.copy()).to(DEV) for a in (v, p, acc0))
    H.hsa_l1_rel_accumulate(tv, tp, ta, False)
    assert np.array_equal(ta.cpu().numpy(), want)
    assert torch.equal(tp, tv)
    H.hsa_l1_rel_accumulate(tv, tp, ta, False)  # no change since: 0/0 adds NaN, 0/x nothing
    want[0] = np.nan
    assert np.array_equal(ta.cpu().numpy(), want, equal_nan=True)
    tp.zero_()
    H.hsa_l1_rel_accumulate(tv, tp, ta, True)
    assert torch.count_nonzero(ta) == 0 and torch.equal(tp, tv)


@pytest.mark.parametrize("shift", [(1, 0), (0, 1)])
def test_l1_rel_off_the_16_byte_alignment(shift):
    """Either array off the 16-byte alignment takes the scalar kernel: the same bits as the vector kernel's."""
    g = _gen(7)
    n, c = 100, 64
    v, p = torch.randn(n, c, generator=g).to(DEV), torch.randn(n, c, generator=g).to(DEV)
    tv, tp = (torch.empty(n * c + 1, device=DEV)[o:o + n * c].view(n, c).copy_(t) for t, o in zip((v, p), shift))
    acc, tacc = torch.zeros(n, dtype=torch.float64, device=DEV), torch.zeros(n, dtype=torch.float64, device=DEV)
    H.hsa_l1_rel_accumulate(v, p, acc, False)
    H.hsa_l1_rel_accumulate(tv, tp, tacc, False)
    assert torch.equal(acc, tacc) and torch.equal(tp, v)


def test_l1_rel_of_the_most_tokens():
    """2^31 - 1 tokens of 8 channels (155 GB): more threads than one launch of the vector kernel may have."""
    n = 2 ** 31 - 1
    if torch.cuda.mem_get_info()[0] < 170 << 30:
        pytest.skip("needs 170 GB of device memory")
    v, p = torch.empty(n, 8, device=DEV), torch.empty(n, 8, device=DEV)
    acc = torch.empty(n, dtype=torch.float64, device=DEV)
    rows = [0, n // 2, n - 1]
    for r in rows:
        v[r], p[r], acc[r] = 2.0, 1.0, 0.25
    H.hsa_l1_rel_accumulate(v, p, acc, False)
    assert acc[rows].tolist() == [0.75] * 3 and bool((p[rows] == 2.0).all())
    del v, p, acc
    torch.cuda.empty_cache()


# one shape per tiling of the bf16 product on 256 compute units (64 x 64, 64 x 128, 128 x 128, 256 x 128,
# 256 x 192, 256 x 256, and 256 x 256 with a split last round whose tiles of the last columns have a ragged
# second half or one past the columns), all with ragged last rows and columns, for the fp32 output too
GEMM_SHAPES = [(65, 68), (1000, 1532), (2000, 1532), (4090, 1532), (8190, 1532), (2590, 5116), (8190, 5116),
               (8190, 4988)]


# K steps 1 .. 8: the large tilings' one and two steps without a loop, the ends of the loops unrolled by 4 and 6
@pytest.mark.parametrize("m,n", GEMM_SHAPES)
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 6, 7, 8])
def test_linear_bf16_edges(m, n, steps):
    g = torch.Generator(device=DEV).manual_seed(m + n + steps)
    k = 64 * steps
    x = torch.randn(m, k, generator=g, device=DEV).to(torch.bfloat16)
    w = (torch.randn(n, k, generator=g, device=DEV) * k ** -0.5).to(torch.bfloat16)
    r = torch.randn(m, n, generator=g, device=DEV).to(torch.bfloat16)
    y = torch.full((m + 1, n), 7.0, device=DEV, dtype=torch.bfloat16)
    H.hsa_linear(x, m, w, y, residual=r)
    want = x.float() @ w.float().t() + r.float()
    # one rounding to bf16 of a value that carries a few fp32 ulps of its terms
    err = (y[:m].float() - want).abs()
    assert bool((err <= 2.0 ** -8 * want.abs() + 1e-5).all())
    assert bool((y[m] == 7.0).all())
    f = torch.full((m + 1, n), 7.0, device=DEV)
    H.hsa_linear(x, m, w, f)
    assert float((f[:m] - (want - r.float())).abs().max()) < 1e-4
    assert bool((f[m] == 7.0).all())


# 64 x 64, the same, 64 x 128, 128 x 128 and, one of the large tilings, 256 x 192 on 256 compute units
@pytest.mark.parametrize("m,d", [(70, 64), (300, 256), (250, 1536), (700, 1536), (2000, 1536)])
def test_qkv_bf16_small_tilings_scatter(m, d):
    """Gathered rows in, scattered rows out, on the small tilings (and a large one); other cache rows untouched."""
    g = torch.Generator(device=DEV).manual_seed(m + d)
    n = 2 * m + 5
    x = torch.randn(n, d, generator=g, device=DEV).to(torch.bfloat16)
    ws = [(torch.randn(d, d, generator=g, device=DEV) * d ** -0.5).to(torch.bfloat16) for _ in range(3)]
    idx = torch.sort(torch.randperm(n, generator=g, device=DEV)[:m]).values.to(torch.int32)
    q = torch.empty(m, d, device=DEV, dtype=torch.bfloat16)
    kc, vc = (torch.full((n, d), 7.0, device=DEV, dtype=torch.bfloat16) for _ in range(2))
    H.hsa_qkv_scatter(x, idx, m, *ws, q, kc, vc)
    rows = x[idx.long()].float()
    for out, w in ((q, ws[0]), (kc[idx.long()], ws[1]), (vc[idx.long()], ws[2])):
        want = rows @ w.float().t()
        assert bool(((out.float() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all())
    skipped = torch.ones(n, dtype=torch.bool, device=DEV)
    skipped[idx.long()] = False
    assert bool((kc[skipped] == 7.0).all()) and bool((vc[skipped] == 7.0).all())


# queries around the small kernel's 16 of a workgroup and the large one's 32 of a wave and 256 of a
# workgroup, rows around the 16-key tiles, the 32-key blocks and the large kernel's 96-row LDS tiles; the
# launcher gives all but (700, 77, 12) and, with a scratch, (40, 3000, 1) to the small kernel
@pytest.mark.parametrize("n_q,n_kv,heads,dh", [
    (1, 1, 1, 128), (15, 15, 2, 64), (16, 17, 2, 128), (17, 31, 1, 128), (33, 95, 2, 128), (255, 97, 1, 64),
    (257, 193, 3, 128), (300, 400, 2, 64), (500, 1000, 2, 128), (40, 3000, 1, 128), (700, 77, 12, 128),
])
@pytest.mark.parametrize("spread", [1.0, 12.0])
@pytest.mark.parametrize("kernel", ["launcher", "large"])
def test_attention_bf16_edges(n_q, n_kv, heads, dh, spread, kernel, monkeypatch):
    """With and without a scratch for key parts; spread 12: the reference maximum has to be raised."""
    if kernel == "large":
        monkeypatch.setenv("HSA_ATTN_WAVES", "8")
    g = _gen(n_q * 1000 + n_kv)
    d = heads * dh
    q, k, v = ((torch.randn(n, d, generator=g) * s).to(torch.bfloat16)
               for n, s in ((n_q, spread), (n_kv, 1.0), (n_kv, 1.0)))
    want = _attend64(q, k, v, heads)
    tq, tk, tv = (t.to(DEV) for t in (q, k, v))
    parts = torch.empty(4 * n_q * heads * (dh + 2) * 4, dtype=torch.uint8, device=DEV)
    # q rescaled and rounded to bf16 moves a score s by up to 2^-8 |s|, which is its probability's
    # relative error (random signs over dh products: a few sigma of s 2^-9 / sqrt(dh) each); p and o
    # round once each
    bar = 2.0 ** -7 * (1 + 0.5 * spread)
    for scratch in (None, parts):
        out = torch.full((n_q + 1, d), 7.0, device=DEV, dtype=torch.bfloat16)
        H.hsa_attention_core(tq, tk, tv, n_q, heads, dh, dh ** -0.5, out, parts=scratch)
        assert float((out[:n_q].cpu().double() - want).abs().max() / want.abs().max()) < bar
        assert bool((out[n_q] == 7.0).all())


@pytest.mark.parametrize("rows,heads,ffn,channels", [(80, 2, 256, 64), (1000, 2, 512, 64), (700, 12, 1536, 64)])
def test_iteration_small_tilings_form_the_rms_factors(rows, heads, ffn, channels):
    """One bf16 layer whose products run on the small tilings, which form the rows' RMS factors themselves,
    against the same calls with hsa_row_rms_scale and its factors."""
    from paper_2605_06892_amd import stack

    g = torch.Generator(device=DEV).manual_seed(rows)
    bf, d = torch.bfloat16, heads * 128
    rn = lambda o, i: (torch.randn(o, i, generator=g, device=DEV) * i ** -0.5).to(bf)  # noqa: E731
    b = stack.StackBuffers.allocate(rows, channels, 0, heads, 128, bf)
    b.x = torch.randn(rows, channels, generator=g, device=DEV)
    b.v_hat = torch.randn(rows, channels, generator=g, device=DEV)
    b.budget.fill_(4)
    b.w_embed, b.w_head = rn(d, channels), rn(channels, d)
    b.layers = [tuple(rn(d, d) for _ in range(4))]
    b.caches = [(torch.zeros(rows, d, device=DEV, dtype=bf), torch.zeros(rows, d, device=DEV, dtype=bf))]
    b.ffn = [(rn(ffn, d), rn(d, ffn))]
    b.f = torch.empty(rows, ffn, device=DEV, dtype=bf)
    xa = b.x.to(bf)
    stack.iteration(b, 4, 1, np.array([1, 0.75, 0.5, 0.25, 0], np.float32))

    h = torch.empty(rows, d, device=DEV, dtype=bf)
    H.hsa_linear(xa, rows, b.w_embed, h)
    scale = torch.empty(rows, device=DEV)
    out = lambda n: torch.empty(rows, n, device=DEV, dtype=bf)  # noqa: E731

    def rms_linear(w, y, **kw):
        H.hsa_row_rms_scale(h, rows, scale)
        H.hsa_linear(h, rows, w, y, row_scale=scale, **kw)
        return y

    wq, wk, wv, wo = b.layers[0]
    q, k, v, o = (rms_linear(w, out(d)) for w in (wq, wk, wv, wv))
    H.hsa_attention_core(q, k, v, rows, heads, 128, 128 ** -0.5, o, parts=b.attn_parts)
    H.hsa_linear(o, rows, wo, h, residual=h)
    f = rms_linear(b.ffn[0][0], out(ffn), gelu=True)
    H.hsa_linear(f, rows, b.ffn[0][1], h, residual=h)
    vel = torch.empty(rows, channels, device=DEV)
    rms_linear(b.w_head, vel)
    # the factors differ in the last bits of their sums only, so K and V by single bf16 roundings
    for got, want in zip(b.caches[0], (k, v)):
        assert bool(((got.float() - want.float()).abs() <= 2.0 ** -7 * want.float().abs() + 1e-6).all())
        assert float((got != want).float().mean()) < 0.01
    # each later layer rounds to bf16 what such a difference moved
    for got, want in ((b.h, h), (b.v_hat, vel)):
        assert float((got.float() - want.float()).norm() / want.float().norm()) < 2.0 ** -7


# 1000 tokens, the first n_lead of them below the full budget: products of 1000 and 1000 - n_lead rows on the
# 64 x 64 (2 heads) and the 64 x 64, 64 x 128 and 128 x 128 tilings (6 heads), and, but for 1000 queries of 6 heads,
# the small attention kernel, whose waves take the 32-key blocks in turn; extra moves the split into other waves' shares
@pytest.mark.parametrize("heads", [2, 6])
@pytest.mark.parametrize("n_lead,extra", [(0, 0), (100, 0), (100, 64), (500, 0), (500, 192), (750, 0)])
def test_prefix_cache_on_the_small_kernels(heads, n_lead, extra):
    """Two bf16 layers with RoPE: keys and values split into a cache prefix and a fresh tail, in the products' stores
    and in the attention's loads, give the bits that a cache of all rows gives; and the first layer's
    cached values are those of its input."""
    from paper_2605_06892_amd import stack

    n, c, d, bf, T = 1000, 64, heads * 128, torch.bfloat16, 8
    sigmas = np.linspace(1, 0, T + 1).astype(np.float32)
    runs = []
    for n_cached in (None, stack.prefix_rows(n_lead, n) + extra):
        g = torch.Generator(device=DEV).manual_seed(heads + n_lead)
        rn = lambda o, i: (torch.randn(o, i, generator=g, device=DEV) * i ** -0.5).to(bf)  # noqa: E731
        b = stack.StackBuffers.allocate(n, c, 2, heads, 128, bf, n_cached=n_cached)
        b.x, b.v_hat = torch.randn(n, c, generator=g, device=DEV), torch.zeros(n, c, device=DEV)
        b.w_embed, b.w_head = rn(d, c), rn(c, d)
        b.layers = [tuple(rn(d, d) for _ in range(4)) for _ in range(2)]
        b.budget.fill_(T)
        b.budget[:n_lead] = torch.tensor([2, 4], dtype=torch.int32, device=DEV)[torch.arange(n_lead, device=DEV) % 2]
        b.enable_rope((2, 20, 25))
        x0 = b.x.to(bf).float()
        # all tokens, those of the full budget, and these with the half budget's
        assert [stack.iteration(b, T, i, sigmas)[0] for i in range(3)] == [n, n - n_lead, n - n_lead // 2 - n_lead % 2]
        runs.append(b)
    full, pre = runs
    rows = pre.n_cached
    assert torch.equal(full.x, pre.x) and torch.equal(full.v_hat, pre.v_hat)
    for (k0, v0), (k1, v1) in zip(full.caches, pre.caches):
        assert torch.equal(k0[:rows], k1[:rows]) and torch.equal(v0[:rows], v1[:rows])
    assert torch.equal(full.caches[-1][0][rows:], pre.k_tail) and torch.equal(full.caches[-1][1][rows:], pre.v_tail)
    # tokens of budget 2 were active in the first iteration only, with x0 as their input
    first = torch.arange(0, n_lead, 2, device=DEV)
    h = (x0[first] @ full.w_embed.float().t()).to(bf).float()
    normed = h * torch.rsqrt((h * h).mean(1, keepdim=True) + 1e-6)
    want = normed @ full.layers[0][2].float().t()
    got = pre.caches[0][1][first].float()
    # two roundings to bf16, of h (summed in another order) and of the value
    assert got.numel() == 0 or float((got - want).norm() / want.norm()) < 2.0 ** -8


@pytest.mark.parametrize("rows,heads", [(80, 2), (300, 40)])
def test_rms_factors_of_the_small_tilings_against_float64(rows, heads):
    """The fp32 velocities of a stack without layers, rms(h) W^T: per row, the factor by which they miss the float64
    product of the same h is on average no larger than with the factors of hsa_row_rms_scale."""
    from paper_2605_06892_amd import stack

    g = torch.Generator(device=DEV).manual_seed(rows)
    bf, d, c = torch.bfloat16, heads * 128, 64
    b = stack.StackBuffers.allocate(rows, c, 0, heads, 128, bf)
    b.x, b.v_hat = torch.randn(rows, c, generator=g, device=DEV), torch.zeros(rows, c, device=DEV)
    b.budget.fill_(4)
    b.w_embed = (torch.randn(d, c, generator=g, device=DEV) * c ** -0.5).to(bf)
    b.w_head = (torch.randn(c, d, generator=g, device=DEV) * d ** -0.5).to(bf)
    stack.iteration(b, 4, 1, np.array([1, 0.75, 0.5, 0.25, 0], np.float32))
    h = b.h[:rows].double()
    want = h * torch.rsqrt((h * h).mean(1, keepdim=True) + 1e-6) @ b.w_head.double().t()
    scale, separate = torch.empty(rows, device=DEV), torch.empty(rows, c, device=DEV)
    H.hsa_row_rms_scale(b.h, rows, scale)
    H.hsa_linear(b.h, rows, b.w_head, separate, row_scale=scale)
    miss = [float(((v.double() * want).sum(1) / (want * want).sum(1) - 1).abs().mean()) for v in (b.v_hat, separate)]
    # a quarter for chance: means over some hundred rows of roundings that both kernels draw alike
    assert miss[0] < 1.25 * miss[1] < 2.0 ** -22


@pytest.mark.parametrize("pinned", [True, False])
@pytest.mark.parametrize("slot", [0, 3, 7])
@pytest.mark.parametrize("n", [1, 5000, 32760])
def test_active_set_count_into_host_memory(pinned, slot, n):
    """The count lands in its own element of a host buffer, inside pinned memory (written by the
    kernel) as in pageable memory (copied), and nowhere else."""
    budget = torch.tensor([8, 4], dtype=torch.int32)[torch.arange(n) % 2].to(DEV)  # iteration 1: the 8s
    idx, count = torch.empty(n, dtype=torch.int32, device=DEV), torch.empty(1, dtype=torch.int32, device=DEV)
    host = torch.full((8,), -77, dtype=torch.int32, pin_memory=pinned)
    want = (n + 1) // 2
    assert H.hsa_build_active_set(budget, 8, 1, 0, idx, count, host_buf=host[slot:]) == want
    assert host.tolist() == [want if i == slot else -77 for i in range(8)]
    assert int(count) == want and torch.equal(idx[:want].cpu(), torch.arange(0, n, 2, dtype=torch.int32))


@pytest.mark.parametrize("inside", ["budget", "idx"])
def test_active_set_count_inside_the_calls_own_arrays(inside):
    """Budgets and indices in pinned memory with the host's count one of their elements: all of them are read and
    written before the count lands."""
    n = 32760
    budget = torch.tensor([8, 4], dtype=torch.int32)[torch.arange(n) % 2].pin_memory()
    idx = torch.full((n,), -7, dtype=torch.int32, pin_memory=True)
    count = torch.empty(1, dtype=torch.int32, device=DEV)
    array, slot = {"budget": (budget, 3), "idx": (idx, 5)}[inside]
    st = H.lib().hsa_build_active_set(budget.data_ptr(), n, 8, 1, 0, idx.data_ptr(), count.data_ptr(),
                                      array[slot:].data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == 0
    want = torch.arange(0, n, 2, dtype=torch.int32)
    if inside == "idx":
        want[slot] = n // 2
    assert torch.equal(idx[:n // 2], want) and bool((idx[n // 2:] == -7).all())
    assert int(count) == n // 2 and int(array[slot]) == n // 2


def test_current_stream_of_the_binding(monkeypatch):
    """The binding's handle of the current stream is torch's, inside and outside a stream's context."""
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert H._stream(None) == torch.cuda.current_stream().cuda_stream == side.cuda_stream
    assert H._stream(None) == torch.cuda.current_stream().cuda_stream
    monkeypatch.setattr(H, "_raw_stream", None)
    assert H._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert H._stream(None) == side.cuda_stream
