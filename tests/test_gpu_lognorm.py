"""The full-vocabulary normaliser on split operands against float64: row
counts at the edges of its kernels (up to 64, 128, 256 rows and chunks of 256),
vocabularies around a tile of 208 words, K from two steps up, and values outside
the split's range, where a tile computes itself again in fp32. A logit's error
is within S (3 x 2^-22 + (3 H / 32 + 4) 2^-24), S = max over words of sum |u| |h|
(three fp16 products per fp32 one, fp32 sums); the sums of exponentials and the
result add a few units in the last place of fp32."""
import numpy as np
import pytest
import torch

from paper_1801_09866_amd import rnnlm as R

pytestmark = pytest.mark.gpu


def data(V, H, n, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return r(V, H) * 0.05, r(V) * 0.05, torch.tanh(r(n, H)) * 0.9


def check(U, b, h):
    got = R.log_normalizer_static(U, b, h)
    torch.cuda.synchronize()
    H = U.shape[1]
    want = torch.logsumexp(h.double() @ U.double().t() + b.double(), dim=1)
    S = (h.double().abs() @ U.double().abs().t()).amax(1)
    bound = S * (3 * 2.0 ** -22 + (3 * H / 32 + 4) * 2.0 ** -24) + 2e-6 + 4 * 2.0 ** -24 * want.abs()
    err = (got.double() - want).abs()
    assert bool((err <= bound).all()), (float(err.max()), float((err / bound).max()))
    return float(err.max())


@pytest.mark.parametrize("n", [1, 15, 16, 17, 48, 64, 65, 96, 128, 129, 200, 255, 256, 257, 321])
@pytest.mark.parametrize("V,H", [(1, 64), (207, 64), (208, 192), (209, 1024), (5000, 2048)])
def test_edges(V, H, n):
    assert check(*data(V, H, n)) < 3e-6   # what fp32 sums show here


@pytest.mark.parametrize("us,hs", [(1e3, 1.0), (1e-5, 1.0), (1e-12, 1e-12), (1.0, 30.0), (1.0, 1e-8), (0.0, 1.0), (1.0, 0.0),
                                   (1e5, 1e-5)])
@pytest.mark.parametrize("n", [5, 100, 256])
def test_scales(us, hs, n):
    U, b, h = data(1000, 128, n)
    check(U * us, b, h * hs)


@pytest.mark.parametrize("n", [3, 256])
def test_one_tile_out_of_range(n):
    """Only the tile that meets the value recomputes; the others are unchanged:
    without that tile's words, the result is the same to the bit."""
    U, b, h = data(1000, 128, n)
    masked = b.clone()
    masked[416:624] = -1e30   # the words of tile 2
    base = R.log_normalizer_static(U, masked, h).clone()
    U[500, 7] = 100.0
    check(U, b, h)
    assert torch.equal(R.log_normalizer_static(U, masked, h), base)


@pytest.mark.parametrize("n", [3, 256])
def test_non_finite(n):
    U, b, h = data(700, 128, n)
    want = torch.logsumexp(h.double() @ U.double().t() + b.double(), dim=1)
    U2 = U.clone()
    U2[300, 5] = float("nan")
    assert bool(torch.isnan(R.log_normalizer_static(U2, b, h)).all())
    h2 = h.abs()
    U2 = U.clone()
    U2[300] = 0.0
    U2[300, 5] = float("-inf")   # a masked word: its logit is -inf, the others' sum stays
    keep = torch.arange(700, device="cuda") != 300
    want = torch.logsumexp(h2.double() @ U[keep].double().t() + b[keep].double(), dim=1)
    assert float((R.log_normalizer_static(U2, b, h2).double() - want).abs().max()) < 3e-6
    b2 = b.clone()
    b2[300] = float("-inf")
    want = torch.logsumexp(h.double() @ U[keep].double().t() + b[keep].double(), dim=1)
    assert float((R.log_normalizer_static(U, b2, h).double() - want).abs().max()) < 3e-6


@pytest.mark.parametrize("n", [3, 100, 256])
def test_row_0_counts_for_its_own_tile_only(n):
    """Word 0 (sentence start) out of range: the other tiles are unchanged. And
    a tile of tiny values beside an ordinary word 0 keeps its precision."""
    U, b, h = data(1000, 128, n)
    masked = b.clone()
    masked[:208] = -1e30   # the words of tile 0
    base = R.log_normalizer_static(U, masked, h).clone()
    U[0, 7] = 100.0
    assert torch.equal(R.log_normalizer_static(U, masked, h), base)
    U, b, h = data(209, 128, n)
    b[:208] = -1e30
    b[208] = 0.0
    U[208] *= 1e-7   # the only word that counts: the result is its logit
    got = R.log_normalizer_static(U, b, h).double()
    want = h.double() @ U[208].double()
    S = h.double().abs() @ U[208].double().abs()
    assert bool(((got - want).abs() <= S * (3 * 2.0 ** -22 + (3 * 128 / 32 + 4) * 2.0 ** -24)).all())


@pytest.mark.parametrize("big", [5.0, 1e4, 1e30])
@pytest.mark.parametrize("n", [3, 64, 65, 100, 200, 256])
def test_one_row_out_of_range(n, big):
    """A history beyond the split's fixed range has a scale of its own, beside
    ordinary and tiny ones."""
    U, b, h = data(1000, 128, n)
    h[n // 2] *= big
    h[n // 2 - 1] *= 1e-9
    check(U, b, h)


@pytest.mark.parametrize("n", [3, 100, 256])
def test_unequal_words_of_a_tile(n):
    """Words far above and far below the fixed range in one tile, rows alike."""
    U, b, h = data(1000, 128, n)
    U *= torch.logspace(-20, 3, 1000, device="cuda")[torch.randperm(1000, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))][:, None]
    h *= torch.logspace(-6, 1, n, device="cuda")[:, None]
    check(U, b, h)


@pytest.mark.parametrize("n", [3, 64, 100, 256])
@pytest.mark.parametrize("value", [float("inf"), float("-inf")])
def test_infinite_row(n, value):
    """A row with an infinity: -inf where it takes every logit there, else NaN
    (two logits of +inf, or infinities of both signs), as in fp32; the other
    rows are right."""
    U, b, h = data(1000, 128, n)
    base = R.log_normalizer_static(U, b, h).clone()
    i = n // 2
    h[i, 70] = value
    got = R.log_normalizer_static(U, b, h).clone()
    assert bool(torch.isnan(got[i]))
    others = torch.arange(n, device="cuda") != i
    assert float((got - base)[others].abs().max()) < 3e-6
    U[:, 70] = -U[:, 70].abs() * (1 if value > 0 else -1)   # every logit of the row is -inf
    assert float(R.log_normalizer_static(U, b, h)[i]) == float("-inf")
    U[:, 70] = -U[:, 70]                                     # every logit is +inf
    assert bool(torch.isnan(R.log_normalizer_static(U, b, h)[i]))
