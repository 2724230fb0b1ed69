"""The f32 contractions on the bf16 matrix instruction (three bf16 of every value, 128 x 128 tiles): at ragged edges against the oracle, and
where the sum of three bf16 is not the value (infinities, NaN, values that round to an infinity, values near the smallest
numbers), against the same product in float64."""
import numpy as np
import pytest
import torch

from oracle import sparse
from paper_2510_11370_amd import r3, synth
from util import Case, assert_close, host, layer_64

pytestmark = pytest.mark.gpu
SH = synth.LayerShape
# every launch of both directions but dH takes split tiles here (of 128 and, down projection, 64): cut on every side, a few hundred to two thousand rows an expert
SPLIT = SH(T=2201, d=500, E=5, K=2, F=580, act="f32", sigma=0.05, zipf_s=0.8, seed=131)


def run(c, calls, dy, x=None):
    w = (c.t["Wg"], c.t["Wu"], c.t["Wd"])
    x = c.t["x"] if x is None else x
    buf = r3.LayerBuffers(c.D, backward=True, gathered_copy=calls == "copy")
    forward = r3.forward_one_call if calls == "one" else r3.forward
    forward(buf, x, c.t["Wr"], c.t["idx"], *w, bias=c.t["bias"])
    r3.backward(buf, dy, x, c.t["Wr"], c.t["idx"], *w)
    torch.cuda.synchronize()
    return buf


def dW_down_64(c, buf, dy):
    """From the H that the layer left (gated by the one-call forward)."""
    off = buf.offsets.tolist()
    tok = buf.perm.long() // c.D.K
    assert buf.gated
    return torch.stack([buf.H[a:b].double().T @ dy[tok[a:b]].double() for a, b in zip(off, off[1:])])


# Of a row's norm.  An f32 chain of 500 to 1000 products leaves 4e-7 to 8e-7 of it, of 2000 1.3e-6, two such in a row 1.1e-6 (dx: from dH); a
# product of pieces that is missing leaves 2.4e-6 (the middle ones with each other) and more.
ROW = 2e-6


def assert_rows(got, want, which=None):
    err, size = (got.double() - want).norm(dim=-1), want.norm(dim=-1)
    if which is not None:
        err, size = err[which], size[which]
        assert (size > 0).all()
    assert (err <= ROW * size).all(), (err / size).max()


@pytest.mark.parametrize("exp", [-104, -112, -118, -122])
def test_small_values_beside_ordinary_ones(exp):
    """Rows and columns whose lowest pieces lie below the smallest bf16 (from 2^-110 down), in tiles of ordinary values."""
    c = Case(SPLIT, backward=True, scale_w=5.0)
    toks = torch.arange(3, SPLIT.T, 50, device="cuda")
    # gradients of a few tokens: dXp
    dy = c.t["dy"].clone()
    dy[toks] *= 2.0 ** exp
    dy[toks + 1] = 0   # (zeros are no small values)
    buf = run(c, "one", dy)
    assert_rows(buf.dx, layer_64(c, buf, dy)["dx"], toks)
    # features of the gradient: dW_down, the other operand
    dy = c.t["dy"].clone()
    cols = torch.arange(5, SPLIT.d, 37, device="cuda")
    dy[:, cols] *= 2.0 ** exp
    buf = run(c, "one", dy)
    assert_rows(buf.dW_down[:, :, cols].transpose(1, 2), layer_64(c, buf, dy)["dW_down"][:, :, cols].transpose(1, 2))
    # a few tokens: SwiGLU; half the exponent: down projection
    for part, e in (("FB", exp), ("Yp", exp / 2)):
        x = c.t["x"].clone()
        x[toks] *= 2.0 ** e
        buf = run(c, "one", c.t["dy"], x)
        rows = torch.isin(buf.perm.long() // SPLIT.K, toks)
        assert_rows({"FB": buf.B, "Yp": buf.Yp}[part], layer_64(c, buf, c.t["dy"], x)[part], rows)


def test_small_columns_behind_zeros():
    """Columns with a few small values within the reduction, zeros around them: some lanes of a wave go through their operand once
    more and others do not.  (The first token's, in two experts that are not looked at, are ordinary.)"""
    c = Case(SPLIT, backward=True, scale_w=5.0)
    cols = torch.arange(5, SPLIT.d, 37, device="cuda")
    dy = c.t["dy"].clone()
    few = torch.arange(500, 1700, 41, device="cuda")
    small = dy[few][:, cols] * 2.0 ** -122
    dy[1:, cols] = 0
    dy[few[:, None], cols] = small
    buf = run(c, "one", dy)
    want = layer_64(c, buf, dy)["dW_down"][:, :, cols].transpose(1, 2)
    without = [e for e in range(SPLIT.E) if e not in c.t["idx"][0].tolist()]
    off = buf.offsets.tolist()
    for e in without:
        tok = (buf.perm[off[e]:off[e + 1]] // SPLIT.K).tolist()
        assert max(tok[:33]) < 500 and min(tok[-33:]) >= 1700
    assert_rows(buf.dW_down[:, :, cols].transpose(1, 2)[without], want[without])


def test_values_without_a_bf16():
    """Every piece of one operand rounds to zero, and what comes out is an ordinary number."""
    c = Case(SPLIT, backward=True, scale_w=1.0)
    dy, x = c.t["dy"] * 2.0 ** -139, c.t["x"] * 2.0 ** 40
    buf = run(c, "one", dy, x)
    want = layer_64(c, buf, dy, x)["dW_down"]
    assert want.abs().max() > 1e-20
    assert (buf.dW_down.double() - want).norm() <= ROW * want.norm()


def test_sums_of_one_and_two_products():
    """Experts of one and two rows among large ones: a product has one rounding, a sum of two no more than one for each."""
    c = Case(SPLIT, backward=True, scale_w=5.0)
    c.t["idx"].copy_(torch.tensor([0, 1]))
    c.t["idx"][1::2] = torch.tensor([1, 2], dtype=torch.uint8, device="cuda")
    c.t["idx"][5] = torch.tensor([0, 3], dtype=torch.uint8, device="cuda")
    c.t["idx"][[9, 1500]] = torch.tensor([2, 4], dtype=torch.uint8, device="cuda")
    dy = c.t["dy"]
    buf = run(c, "one", dy)
    off = buf.offsets.tolist()
    assert [off[4] - off[3], off[5] - off[4]] == [1, 2]
    assert torch.equal(buf.dW_down[3], buf.H[off[3]][:, None] * dy[5][None])
    terms = (buf.H[off[4]:].double()[:, :, None] * dy[[9, 1500]].double()[:, None])
    assert ((buf.dW_down[4].double() - terms.sum(0)).abs() <= 2.0 ** -23 * terms.abs().sum(0)).all()


@pytest.mark.parametrize("calls", ["one", "steps", "copy"])
@pytest.mark.parametrize("sh", [
    SPLIT, SH(T=4100, d=260, E=40, K=2, F=1028, act="f32", sigma=0.05, zipf_s=1.2, seed=132),   # experts of few rows
    SH(T=4100, d=516, E=4, K=2, F=512, act="f32", sigma=0.05, seed=135),                        # tiles of 128 in every launch
    SH(T=130, d=516, E=9, K=2, F=524, act="f32", sigma=0.05, seed=136),                         # tiles of 32
    SH(T=2050, d=132, E=30, K=2, F=388, act="f32", sigma=0.05, seed=137)],                      # narrow: split gradients beside dXp on the f32 instruction
                         ids=lambda s: "T%d_d%d_F%d_E%d" % (s.T, s.d, s.F, s.E))
def test_layer(sh, calls):
    c = Case(sh, backward=True, scale_w=5.0)
    n = c.np
    fwd = sparse.forward(n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], n["bias"])
    ref = sparse.backward(n["dy"], n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], fwd)
    buf = run(c, calls, c.t["dy"])
    # each contraction by itself, row by row
    want = layer_64(c, buf, c.t["dy"])
    for name, got in (("FA", buf.A), ("FB", buf.B), ("Yp", buf.Yp), ("dx", buf.dx), ("dW_gate", buf.dW_gate), ("dW_up", buf.dW_up), ("dW_down", buf.dW_down)):
        assert_rows(got, want[name])
    # f32 sums of up to 2000 terms, up to three in a row: an f32 FMA chain leaves 1e-6 of the norm here, 4e-6 is four times that
    for got, want in ((buf.y, fwd["y"]), (buf.dx, ref["dx"]), (buf.dW_gate, ref["dWg"]), (buf.dW_up, ref["dWu"]), (buf.dW_down, ref["dWd"])):
        got = host(got).astype(np.float64)
        assert np.linalg.norm(got - want) <= 4e-6 * np.linalg.norm(want)
    assert_close(host(buf.y), fwd["y"], "y", c.rel)
    assert_close(host(buf.dx), ref["dx"], "dx", c.rel)


@pytest.mark.parametrize("what", ["inf", "-inf", "nan", "rounds_to_inf", "tiny", "zero"])
def test_where_three_bf16_are_not_the_value(what):
    c = Case(SPLIT, backward=True, scale_w=1.0)
    dy = c.t["dy"].clone()
    if what == "tiny":
        dy *= 2.0 ** -122
    elif what == "zero":
        dy.zero_()
    else:
        dy[7, 3] = {"inf": np.inf, "-inf": -np.inf, "nan": np.nan, "rounds_to_inf": 3.4e38}[what]
    buf = run(c, "one", dy)
    got, want = buf.dW_down.double(), dW_down_64(c, buf, dy).float().double()
    assert torch.equal(got.isnan(), want.isnan())
    assert torch.equal(got.isinf(), want.isinf()) and torch.equal(got[got.isinf()], want[want.isinf()])
    if what in ("inf", "-inf", "nan"):
        assert not want.isfinite().all()
    f = want.isfinite()
    big = f & (want.abs() > 1e30)
    assert big.any() == (what == "rounds_to_inf")
    for part in (big, f & ~big):
        assert (got - want)[part].norm() <= ROW * want[part].norm()


def test_nan_stays_with_its_token():
    c = Case(SPLIT, backward=True, scale_w=1.0)
    clean = run(c, "one", c.t["dy"]).y.clone()
    x = c.t["x"].clone()
    x[11, 5], x[900, 0] = np.nan, np.inf
    buf = r3.LayerBuffers(c.D, backward=False, gathered_copy=False)
    r3.forward_one_call(buf, x, c.t["Wr"], c.t["idx"], c.t["Wg"], c.t["Wu"], c.t["Wd"], bias=c.t["bias"])
    torch.cuda.synchronize()
    hit = torch.zeros(SPLIT.T, dtype=torch.bool, device="cuda")
    hit[[11, 900]] = True
    assert not buf.y[hit].isfinite().any()
    # the f32 instruction has these tokens' rows, in the tiles of other rows that keep their bits
    assert torch.equal(buf.y[~hit], clean[~hit])


@pytest.mark.parametrize("calls", ["one", "steps"])
@pytest.mark.parametrize("sh", [
    SH(T=4200, d=500, E=5, K=2, F=580, act="f32", sigma=0.05, zipf_s=0.8, seed=133),    # split tiles: of 32, 64 and 128 rows
    SH(T=4200, d=132, E=6, K=2, F=260, act="f32", sigma=0.05, zipf_s=0.8, seed=134),    # f32 instruction: of 32 and 64
    SH(T=4200, d=131, E=6, K=3, F=259, act="f32", sigma=0.05, zipf_s=0.8, seed=138),    # widths that are no multiples of four
], ids=lambda s: "d%d_F%d" % (s.d, s.F))
def test_rows_do_not_depend_on_the_batch(sh, calls):
    """A token's y and dx are the same bits in a micro-batch and in the whole batch."""
    c = Case(sh, backward=True, scale_w=5.0)
    c.t["dy"][::97] *= 2.0 ** -118   # rows that the f32 instruction has, in any tile
    whole = run(c, calls, c.t["dy"])
    for T in (1, 37, 300, 1100, 2900):
        part = Case.__new__(Case)
        part.D = r3.desc(T, sh.d, sh.E, sh.K, sh.F, sh.act)
        part.t = {k: v[:T].contiguous() if k in ("x", "dy", "idx") else v for k, v in c.t.items()}
        buf = run(part, calls, part.t["dy"])
        for name in ("gates", "y", "dx"):
            assert torch.equal(getattr(buf, name), getattr(whole, name)[:T]), (name, T)
