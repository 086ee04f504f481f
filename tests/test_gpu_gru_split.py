"""The fp32 GRU on split operands (each value the sum of two fp16 numbers)
against the same step in float64: row counts at the edges of row blocks, tiles
and unit widths, model widths whose K steps divide unevenly among the waves,
one and two layers, and operands scaled far from 1 or mixed in one row. The
bound per value follows the arithmetic: an operand's two parts miss it by at
most 2^-22 of itself and lo x lo (2^-22) is left out, so a product is within
3 x 2^-22, and the fp32 sums of 3 K / 32 matrix instructions and four partial
sums round by at most 2^-24 of S = sum |w| |a| each. Non-finite weights and
embeddings have no split form; they must give fp32's infinities and NaNs, and
change nothing else."""
import numpy as np
import pytest
import torch

from paper_1801_09866_amd import rnnlm as R
from paper_1801_09866_amd.workload import BF16, F32, ModelCfg

pytestmark = pytest.mark.gpu


def make(E, H, L, sigma=0.05, seed=3, V=300):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda") * sigma
    m = ModelCfg(V=V, E=E, H=H, L=L, wdtype=F32, maxent_log2=4, maxent_order=1)
    w = {"emb": n(V, E), "W_ih": [n(3 * H, E if l == 0 else H) for l in range(L)],
         "W_hh": [n(3 * H, H) for l in range(L)], "b_ih": [n(3 * H) for l in range(L)],
         "U_out": n(V, H), "b_out": n(V), "maxent": n(16)}
    return m, w


def step64(m, w, vec, w1):
    """h' and its error bound, per value, in float64."""
    x, out, bnd = w["emb"][w1].double(), [], []
    dx = torch.zeros_like(x)
    for l in range(m.L):
        H = m.H
        h = vec[:, l * H:(l + 1) * H].double()
        Wi, Wh, b = w["W_ih"][l].double(), w["W_hh"][l].double(), w["b_ih"][l].double()
        gi, gh = x @ Wi.t() + b, h @ Wh.t()
        K = Wi.shape[1] + H
        unit = 3 * 2.0 ** -22 + (3 * K / 32 + 10) * 2.0 ** -24
        # a part's scale follows its own largest value, or the other part's
        # where that is at most 2^8 times as large: what is far below it is off
        # by up to 2^-38 of that. A second layer's input is scaled by its bound.
        own = lambda a, other: 2.0 ** -38 * torch.minimum(torch.maximum(a, other), 256 * a)
        ax, ah = x.abs().amax(1), h.abs().amax(1)
        if l:
            ax = vec[:, :H].double().abs().amax(1).clamp(min=1.0)
        fx, fh = own(ax, ah)[:, None], own(ah, ax)[:, None]
        wi, wh = Wi.abs().amax(1), Wh.abs().amax(1)
        ei = (unit * (x.abs() @ Wi.abs().t() + b.abs()) + dx @ Wi.abs().t() + fx * Wi.abs().sum(1)
              + own(wi, wh) * x.abs().sum(1)[:, None])
        eh = unit * (h.abs() @ Wh.abs().t()) + fh * Wh.abs().sum(1) + own(wh, wi) * h.abs().sum(1)[:, None]
        r, z = torch.sigmoid(gi[:, :H] + gh[:, :H]), torch.sigmoid(gi[:, H:2 * H] + gh[:, H:2 * H])
        n = torch.tanh(gi[:, 2 * H:] + r * gh[:, 2 * H:])
        dr, dz = (ei + eh)[:, :H] / 4, (ei + eh)[:, H:2 * H] / 4
        dn = ei[:, 2 * H:] + eh[:, 2 * H:] + dr * gh[:, 2 * H:].abs()
        hn = (1 - z) * n + z * h
        d = dz * (n.abs() + h.abs()) + dn + 6 * 2.0 ** -24 * (1 + h.abs())
        out.append(hn)
        bnd.append(d)
        x, dx = hn, d
    return torch.cat(out, 1), torch.cat(bnd, 1)


def run(m, w, vec, w1, qmode=R.Q_SIGN, sessions=1, digits=0):
    B = vec.shape[0] // sessions
    sc = R.Scorer(m, w, qmode, digits, max_hist=B, max_query=1, cap_hist=2048, cap_query=16, sessions=sessions)
    words = torch.zeros((vec.shape[0], 3), dtype=torch.int32, device="cuda")
    words[:, 0] = w1.int()
    e = torch.zeros(0, dtype=torch.int32, device="cuda")
    if sessions == 1:
        out = [sc.score_frame(vec, words, e, e)]
    else:
        out = sc.score_frames([(vec[k * B:(k + 1) * B].contiguous(), words[k * B:(k + 1) * B].contiguous(), e, e)
                               for k in range(sessions)])
    torch.cuda.synchronize()
    return torch.cat([o["hnew"] for o in out]), sc.stats()


def rows(M, m, seed=5, scale=0.7):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.tanh(torch.randn(M, m.L * m.H, generator=g, device="cuda")) * scale,
            torch.randint(0, m.V, (M,), generator=g, device="cuda"))


@pytest.mark.parametrize("E,H,L", [(64, 64, 1), (64, 192, 2), (192, 128, 1), (128, 320, 2), (512, 1024, 1), (320, 1024, 2)])
@pytest.mark.parametrize("M", [1, 15, 16, 17, 33, 64, 65, 128, 129, 300, 513])
def test_row_counts_and_widths(E, H, L, M):
    m, w = make(E, H, L)
    vec, w1 = rows(M, m)
    got, st = run(m, w, vec, w1)
    assert st["gru_rows"] == M
    want, bound = step64(m, w, vec, w1)
    err = (got.double() - want).abs()
    assert bool((err <= bound).all()), float((err / bound).max())
    # far inside the bound on ordinary operands: no more than fp32 sums show
    assert float(err.norm() / want.norm()) < 3e-7


@pytest.mark.parametrize("sessions", [2, 8])
def test_sessions_share_the_launch(sessions):
    m, w = make(128, 256, 2)
    vec, w1 = rows(sessions * 45, m)
    got, st = run(m, w, vec, w1, sessions=sessions)
    want, bound = step64(m, w, vec, w1)
    assert bool(((got.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("hscale,escale,wscale", [(1e-30, 1.0, 1.0), (1e-6, 1e-6, 1.0), (1e4, 1.0, 1e-3), (1.0, 1e3, 1e-3),
                                                  (0.0, 1.0, 1.0), (0.0, 0.0, 1.0), (1.0, 1.0, 0.0), (1e30, 1e-30, 1e-30),
                                                  (1.0, 1e-37, 1e-37)])
def test_scales(hscale, escale, wscale):
    m, w = make(128, 128, 2)
    w["emb"] *= escale
    for k in ("W_ih", "W_hh"):
        w[k] = [x * wscale for x in w[k]]
    vec, w1 = rows(40, m)
    vec = vec * hscale
    got, st = run(m, w, vec, w1, qmode=R.Q_SIGN)
    want, bound = step64(m, w, vec, w1)
    assert st["device_error"] == 0
    assert bool(((got.double() - want).abs() <= bound).all()), float(((got.double() - want).abs() / bound).max())


def test_mixed_magnitudes_in_a_row():
    m, w = make(128, 256, 1)
    vec, w1 = rows(70, m)
    vec *= torch.logspace(-12, 0, 256, device="cuda")
    got, _ = run(m, w, vec, w1)
    want, bound = step64(m, w, vec, w1)
    assert bool(((got.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("where", ["emb", "W_ih", "W_hh", "W_hh1"])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_non_finite_operands(where, value):
    """One non-finite value; fp32 sums that meet it are inf or NaN, all others
    as without it."""
    m, w = make(64, 128, 2)
    vec, w1 = rows(37, m)
    w1[3] = 7
    t = {"emb": w["emb"], "W_ih": w["W_ih"][0], "W_hh": w["W_hh"][0], "W_hh1": w["W_hh"][1]}[where]
    t[(7, 5) if where == "emb" else (2 * m.H + 9, 11)] = value
    got, st = run(m, w, vec, w1)
    assert st["device_error"] == 0
    x, ref = w["emb"][w1], []
    for l in range(m.L):
        H = m.H
        h = vec[:, l * H:(l + 1) * H]
        gi = torch.stack([(x * row).sum(1) for row in w["W_ih"][l]], 1) + w["b_ih"][l]
        gh = torch.stack([(h * row).sum(1) for row in w["W_hh"][l]], 1)
        r, z = torch.sigmoid(gi[:, :H] + gh[:, :H]), torch.sigmoid(gi[:, H:2 * H] + gh[:, H:2 * H])
        x = (1 - z) * torch.tanh(gi[:, 2 * H:] + r * gh[:, 2 * H:]) + z * h
        ref.append(x)
    ref = torch.cat(ref, 1)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    ok = ~torch.isnan(ref)
    assert float((got - ref)[ok].abs().max()) < 2e-6


@pytest.mark.parametrize("qmode,digits", [(R.Q_SIGN, 0), (R.Q_SIGDIG, 2)])
@pytest.mark.parametrize("E,H,L", [(64, 64, 1), (192, 64, 2), (64, 320, 2), (576, 128, 1), (512, 1024, 2), (4160, 64, 1),
                                   (64, 2048, 1)])
@pytest.mark.parametrize("M", [1, 16, 17, 64, 65, 129, 512, 513, 1024])
def test_bf16_packed_rows(E, H, L, M, qmode, digits):
    """bf16 models in launches of at most 1024 histories (512 at H = 2048, where
    more take the other kernel): odd and even numbers
    of 64-value lines in either part, rows longer than a thread group reads at
    once. Each layer against float64 on the bf16 operands it really had (the
    second layer's input is the first one's h', rounded), so the bound is that
    of the fp32 sums alone."""
    m, w = make(E, H, L)
    m = ModelCfg(V=m.V, E=E, H=H, L=L, wdtype=BF16, maxent_log2=4, maxent_order=1)
    w = {k: [x.bfloat16() for x in v] if k[0] == "W" else v.bfloat16() if k in ("emb", "U_out") else v for k, v in w.items()}
    vec, w1 = rows(M, m)
    sc = R.Scorer(m, w, qmode, digits, max_hist=M, max_query=1, cap_hist=2048, cap_query=16)
    words = torch.zeros((M, 3), dtype=torch.int32, device="cuda")
    words[:, 0] = w1.int()
    e = torch.zeros(0, dtype=torch.int32, device="cuda")
    out = sc.score_frame(vec, words, e, e)
    torch.cuda.synchronize()
    got = out["hnew"]
    rep = out["h_rep"][:M].long()
    assert int(sc.stats()["gru_rows"]) == int((rep == torch.arange(M, device="cuda")).sum())
    vec, x = vec[rep], w["emb"][w1].double()   # few values at two digits may merge rows
    for l in range(L):
        h = vec[:, l * H:(l + 1) * H]
        hb = h.bfloat16().double()
        Wi, Wh, b = w["W_ih"][l].double(), w["W_hh"][l].double(), w["b_ih"][l].double()
        gi, gh = x @ Wi.t() + b, hb @ Wh.t()
        r, z = torch.sigmoid(gi[:, :H] + gh[:, :H]), torch.sigmoid(gi[:, H:2 * H] + gh[:, H:2 * H])
        n = torch.tanh(gi[:, 2 * H:] + r * gh[:, 2 * H:])
        want = (1 - z) * n + z * h.double()
        unit = ((E if l == 0 else H) + H) / 32 * 2.0 ** -24
        bound = unit * (x.abs() @ Wi.abs().t() + hb.abs() @ Wh.abs().t() + b.abs()).reshape(M, 3, H).sum(1) + 6 * 2.0 ** -24 * (1 + h.abs())
        g = got[:, l * H:(l + 1) * H]
        err = (g.double() - want).abs()
        assert bool((err <= bound).all()), (l, float((err / bound).max()))
        x = g.bfloat16().double()


def parts_scaled(es, hs, wis, whs, E=128, H=256, M=40):
    m, w = make(E, H, 1)
    w["emb"] *= es
    w["W_ih"][0] *= wis
    w["W_hh"][0] *= whs
    vec, w1 = rows(M, m)
    return m, w, vec * hs, w1


@pytest.mark.parametrize("s,k", [(1e-36, 1.0), (1e30, 1.0), (1e-34, 40.0)])
def test_weights_and_rows_far_apart(s, k):
    """Operands near either end of fp32's range whose sums are not (k: their size)."""
    m, w, vec, w1 = parts_scaled(s, s, k / s, k / s)
    got, _ = run(m, w, vec, w1)
    want, bound = step64(m, w, vec, w1)
    assert bool(((got.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("gate", [0, 1, 2])
@pytest.mark.parametrize("where", ["W_ih", "W_hh", "W_ih1", "W_hh1"])
@pytest.mark.parametrize("value", [30.0, 1e4, 1e6, 1e8])
def test_one_large_weight(where, value, gate):
    """It costs the units that do not use it nothing."""
    m, w = make(128, 256, 2)
    vec, w1 = rows(40, m)
    l = int(where.endswith("1"))
    w[where[:4]][l][gate * m.H + 9, 11] = value
    got, _ = run(m, w, vec, w1)
    want, bound = step64(m, w, vec, w1)
    err = (got.double() - want).abs()
    assert bool((err <= bound).all()), float((err / bound).max())
    others = torch.ones(m.L * m.H, dtype=torch.bool, device="cuda")
    others[l * m.H + 9] = False
    assert float(err[:, others].norm() / want[:, others].norm()) < 3e-7


@pytest.mark.parametrize("es,hs,wis,whs", [(1e-6, 1.0, 1e6, 1.0), (1.0, 1e-6, 1.0, 1e6), (1e-20, 1.0, 1e20, 1.0), (1.0, 1e-20, 1.0, 1e20),
                                           (1e-3, 1.0, 1e3, 1.0), (1.0, 1e-36, 1.0, 1e36), (1e-36, 1.0, 1e36, 1.0), (1.0, 0.0, 1.0, 1.0),
                                           (1.0, 1.0, 1.0, 0.0), (1.0, 1.0, 0.0, 1.0), (0.0, 1.0, 1.0, 1.0), (1.0, 1.0, 1.0, 1e-30),
                                           (1.0, 1e-30, 1.0, 1e-10), (1e-30, 1.0, 1e-10, 1.0)])
@pytest.mark.parametrize("E,H,M", [(64, 64, 5), (128, 256, 40), (512, 1024, 150), (512, 1024, 600)])
def test_input_and_recurrent_parts_of_other_sizes(es, hs, wis, whs, E, H, M):
    """One part's values small, its weights large: its products count as much
    as the other part's, so each part keeps its own precision."""
    m, w, vec, w1 = parts_scaled(es, hs, wis, whs, E, H, M)
    got, _ = run(m, w, vec, w1)
    want, bound = step64(m, w, vec, w1)
    err = (got.double() - want).abs()
    assert bool((err <= bound).all()), float((err / bound).max())
    # what fp32 sums show
    assert float(err.norm() / want.norm()) < 3e-7


def test_packed_rows_beyond_32_bit_offsets():
    """Eight sessions of 2048 histories of 65,600 operands: more packed rows
    than 32-bit offsets reach. Such a model keeps the kernel of exact keys, and
    its results to the bit."""
    m, w = make(65536, 64, 1, V=20)
    vec, w1 = rows(70, m)
    out = {}
    for qmode in (R.Q_SIGN, R.Q_EXACT):
        sc = R.Scorer(m, w, qmode, 0, max_hist=2048, max_query=1, cap_hist=256, cap_query=16, sessions=8)
        words = torch.zeros((70, 3), dtype=torch.int32, device="cuda")
        words[:, 0] = w1.int()
        e = torch.zeros(0, dtype=torch.int32, device="cuda")
        out[qmode] = sc.score_frame(vec, words, e, e)["hnew"].clone()
        torch.cuda.synchronize()
        assert sc.stats()["gru_rows"] == 70
    assert torch.equal(out[R.Q_SIGN], out[R.Q_EXACT])
    want, bound = step64(m, w, vec, w1)
    err = (out[R.Q_SIGN].double() - want).abs()
    # this kernel's sums: one rounding per four products
    bound = bound + (65600 / 4) * 2.0 ** -24 * (1 + want.abs())
    assert bool((err <= bound).all())


@pytest.mark.parametrize("L", [1, 2])
@pytest.mark.parametrize("rows_each", [45, 300])
def test_non_finite_embedding_leaves_the_other_rows(L, rows_each):
    """One session meets a word with a non-finite embedding: no other row of
    either session changes by a bit."""
    m, w = make(64, 192, L)
    vec, w1 = rows(2 * rows_each, m)
    w1[w1 == 7] = 8
    w1[3] = 7
    base, _ = run(m, w, vec, w1, sessions=2)
    w["emb"][7, 5] = float("inf")
    got, _ = run(m, w, vec, w1, sessions=2)
    keep = torch.arange(2 * rows_each, device="cuda") != 3
    assert torch.equal(got[keep], base[keep])
    assert not torch.equal(got[3], base[3])


@pytest.mark.parametrize("where", ["W_ih", "W_hh", "W_hh1"])
@pytest.mark.parametrize("gate", [0, 1, 2])
@pytest.mark.parametrize("M", [5, 150])
def test_non_finite_weight_leaves_the_other_units(where, gate, M):
    m, w = make(64, 192, 2 if where == "W_hh1" else 1)
    vec, w1 = rows(M, m)
    base, _ = run(m, w, vec, w1)
    l = int(where.endswith("1"))
    w[where[:4]][l][gate * m.H + 9, 11] = float("inf")
    got, _ = run(m, w, vec, w1)
    keep = torch.arange(m.L * m.H, device="cuda") != l * m.H + 9
    assert torch.equal(got[:, keep], base[:, keep])


@pytest.mark.parametrize("qmode,digits", [(R.Q_SIGN, 0), (R.Q_SIGDIG, 2)])
@pytest.mark.parametrize("E,H,L", [(576, 128, 1), (1088, 64, 2), (4160, 64, 1), (128, 1024, 2)])
@pytest.mark.parametrize("M", [1, 17, 129, 300])
def test_key_modes_and_long_embeddings(E, H, L, M, qmode, digits):
    """Rows packed by a wave and by a block; embeddings longer than what either reads before its cache probe."""
    m, w = make(E, H, L)
    vec, w1 = rows(M, m)
    got, st = run(m, w, vec, w1, qmode=qmode, digits=digits)
    assert st["gru_rows"] == M
    want, bound = step64(m, w, vec, w1)
    err = (got.double() - want).abs()
    assert bool((err <= bound).all()), float((err / bound).max())
    assert float(err.norm() / want.norm()) < 3e-7
