"""The bf16 expert GEMMs at widths that are multiples of 8 but not of their 256 x 256 tiles: reductions that end inside a
64-k window, feature tiles that end inside a wave's share, tail row tiles, and split weight-gradient reductions.  Both
forwards and their backward against the CPU oracle, with the bars of tests/util.py."""
import numpy as np
import pytest
import torch

from oracle import sparse
from paper_2510_11370_amd import r3, synth
from util import Case, assert_close, host, router_gradient_sigma

pytestmark = pytest.mark.gpu
SH = synth.LayerShape


@pytest.mark.parametrize("sh,one_call", [
    (SH(T=300, d=264, E=128, K=8, F=136, sigma=0.02, seed=71), True),        # 8 over a window / a tile
    (SH(T=611, d=504, E=16, K=6, F=328, sigma=0.02, zipf_s=1.0, seed=72), True),
    (SH(T=611, d=504, E=16, K=6, F=328, sigma=0.02, zipf_s=1.0, seed=72), False),
    (SH(T=77, d=1000, E=60, K=4, F=704, sigma=0.02, seed=73), True),         # tail tiles only
    (SH(T=3000, d=256, E=16, K=2, F=72, sigma=0.02, seed=74), False),        # one width whole, the other not
    (SH(T=9216, d=264, E=128, K=4, F=264, sigma=0.02, zipf_s=2.5, seed=75), True),   # split reductions
], ids=lambda v: ("T%d_d%d_F%d" % (v.T, v.d, v.F)) if isinstance(v, SH) else ("one" if v else "steps"))
def test_layer_at_ragged_widths(sh, one_call):
    c = Case(sh, backward=True, scale_w=5.0)
    n = c.np
    fwd = sparse.forward(n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], n["bias"])
    ref = sparse.backward(n["dy"], n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], fwd, want_dbias=True)
    w = (c.t["Wg"], c.t["Wu"], c.t["Wd"])
    buf = r3.LayerBuffers(c.D, backward=True, gathered_copy=not one_call)
    for t in (buf.Yp, buf.H, buf.A, buf.B, buf.dx, buf.dW_gate, buf.dW_up, buf.dW_down):
        t.fill_(7.0)      # an element left unwritten, or written past its row, shows
    (r3.forward_one_call if one_call else r3.forward)(buf, c.t["x"], c.t["Wr"], c.t["idx"], *w, bias=c.t["bias"])
    r3.backward(buf, c.t["dy"], c.t["x"], c.t["Wr"], c.t["idx"], *w)
    torch.cuda.synchronize()
    assert int(buf.status.item()) == 0
    g = fwd["g"].reshape(-1)[fwd["perm"]][:, None] if one_call else 1.0
    assert_close(host(buf.H), g * fwd["h"], "H", c.rel)
    assert_close(host(buf.Yp), g * fwd["o"], "Yp", c.rel)
    assert_close(host(buf.y), fwd["y"], "y", c.rel)
    assert_close(host(buf.dx), ref["dx"], "dx", c.rel)
    assert_close(buf.dW_r.cpu().numpy(), ref["dWr"], "dW_r", c.rel,
                 router_gradient_sigma(n["x"], n["dy"], c.idx, fwd, sh.E)[0])
    for got, key in ((buf.dW_gate, "dWg"), (buf.dW_up, "dWu"), (buf.dW_down, "dWd")):
        got = got.cpu().numpy()
        for e in range(sh.E):
            assert np.linalg.norm(got[e] - ref[key][e]) <= c.rel * np.linalg.norm(ref[key][e]) + 1e-30, (key, e)
    # added to instead of overwritten: twice the gradient (a sum of two f32, in parts where a reduction is split)
    grads = (buf.dW_r, buf.dW_gate, buf.dW_up, buf.dW_down)
    once = [t.double() for t in grads]
    r3.backward(buf, c.t["dy"], c.t["x"], c.t["Wr"], c.t["idx"], *w, accumulate=True)
    torch.cuda.synchronize()
    for t, o in zip(grads, once):
        assert float((t.double() - 2 * o).norm()) <= 1e-6 * float((2 * o).norm())
    # a caller that gives Xp need not give perm, nor fill one: every output again
    if not one_call:
        sigma = router_gradient_sigma(n["x"], n["dy"], c.idx, fwd, sh.E)
        for perm in (None, torch.zeros_like(buf.perm)):
            dbias = torch.full((sh.E,), 3.0, dtype=torch.float32, device="cuda")
            for t in (buf.dx, buf.dW_r, buf.dW_gate, buf.dW_up, buf.dW_down):
                t.fill_(7.0)
            r3.moe_backward(buf.D, c.t["dy"], c.t["x"], c.t["Wr"], c.t["idx"], buf.gates, buf.inv_perm, perm, buf.offsets,
                            buf.Xp, buf.A, buf.B, buf.H, buf.Yp, *w, buf.dx, buf.dW_r, buf.dW_gate, buf.dW_up, buf.dW_down,
                            buf.ws_bwd, dbias=dbias)
            torch.cuda.synchronize()
            assert_close(dbias.cpu().numpy(), ref["dbias"], "dbias without perm", c.rel, sigma[1])
            assert_close(buf.dW_r.cpu().numpy(), ref["dWr"], "dW_r without perm", c.rel, sigma[0])
            assert_close(host(buf.dx), ref["dx"], "dx without perm", c.rel)
            for got, key in ((buf.dW_gate, "dWg"), (buf.dW_up, "dWu"), (buf.dW_down, "dWd")):
                got = got.cpu().numpy()
                for e in range(sh.E):
                    assert np.linalg.norm(got[e] - ref[key][e]) <= c.rel * np.linalg.norm(ref[key][e]) + 1e-30, (key, e)


@pytest.mark.parametrize("d,F", [(256, 256), (320, 192)])     # whole tiles; guarded ones, five and three windows of 64 k
def test_rows_per_expert_at_tile_edges(d, F):
    """Experts with 0, 1, 64, 65, 128, 129, 192, 256, 257 and 385 rows: every loop a row tile can take, and its edges."""
    rows = [0, 1, 64, 65, 128, 129, 192, 256, 257, 385]
    sh = SH(T=sum(rows), d=d, E=len(rows), K=1, F=F, seed=76)
    c = Case(sh, backward=True, scale_w=5.0)
    c.idx = np.random.default_rng(0).permutation(np.repeat(np.arange(len(rows)), rows)).astype(np.int32)[:, None]
    c.t["idx"] = torch.from_numpy(c.idx.astype(np.uint8)).to("cuda")
    n = c.np
    fwd = sparse.forward(n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], n["bias"])
    ref = sparse.backward(n["dy"], n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], fwd, want_dbias=True)
    w = (c.t["Wg"], c.t["Wu"], c.t["Wd"])
    buf = r3.LayerBuffers(c.D, backward=True, gathered_copy=False)
    for t in (buf.Yp, buf.H, buf.A, buf.B, buf.dx):
        t.fill_(7.0)
    r3.forward_one_call(buf, c.t["x"], c.t["Wr"], c.t["idx"], *w, bias=c.t["bias"])
    r3.backward(buf, c.t["dy"], c.t["x"], c.t["Wr"], c.t["idx"], *w)
    torch.cuda.synchronize()
    assert buf.counts.tolist() == rows
    for got, want, name in ((buf.H, fwd["h"], "H"), (buf.Yp, fwd["o"], "Yp"), (buf.y, fwd["y"], "y"), (buf.dx, ref["dx"], "dx")):
        assert_close(host(got), want, name, c.rel)
    for got, key in ((buf.dW_gate, "dWg"), (buf.dW_up, "dWu"), (buf.dW_down, "dWd")):
        got = got.cpu().numpy()
        for e in range(sh.E):
            assert np.linalg.norm(got[e] - ref[key][e]) <= c.rel * np.linalg.norm(ref[key][e]) + 1e-30, (key, e)


@pytest.mark.parametrize("one_call", [True, False])
@pytest.mark.parametrize("d,F", [(256, 512), (264, 136)])     # whole tiles; guarded ones
def test_tail_tiles(d, F, one_call):
    """Row tiles of at most 128 rows, whose rows and features all eight waves share: at the edges of a wave's 16- and 32-row blocks
    and of the two arrangements, alone and behind a full tile."""
    rows = [15, 16, 17, 31, 32, 33, 48, 63, 95, 96, 97, 127, 256 + 32, 256 + 33, 256 + 96, 256 + 97]
    sh = SH(T=sum(rows), d=d, E=len(rows), K=1, F=F, seed=78)
    c = Case(sh, backward=True, scale_w=5.0)
    c.idx = np.random.default_rng(1).permutation(np.repeat(np.arange(len(rows)), rows)).astype(np.int32)[:, None]
    c.t["idx"] = torch.from_numpy(c.idx.astype(np.uint8)).to("cuda")
    n = c.np
    fwd = sparse.forward(n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], n["bias"])
    ref = sparse.backward(n["dy"], n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], fwd, want_dbias=True)
    w = (c.t["Wg"], c.t["Wu"], c.t["Wd"])
    buf = r3.LayerBuffers(c.D, backward=True, gathered_copy=False)
    for t in (buf.Yp, buf.H, buf.A, buf.B, buf.dx):
        t.fill_(7.0)
    (r3.forward_one_call if one_call else r3.forward)(buf, c.t["x"], c.t["Wr"], c.t["idx"], *w, bias=c.t["bias"])
    r3.backward(buf, c.t["dy"], c.t["x"], c.t["Wr"], c.t["idx"], *w)
    torch.cuda.synchronize()
    assert buf.counts.tolist() == rows
    for got, want, name in ((buf.H, fwd["h"], "H"), (buf.Yp, fwd["o"], "Yp"), (buf.y, fwd["y"], "y"), (buf.dx, ref["dx"], "dx")):
        assert_close(host(got), want, name, c.rel)      # (one expert per token: the gate is 1)
    for got, key in ((buf.dW_gate, "dWg"), (buf.dW_up, "dWu"), (buf.dW_down, "dWd")):
        got = got.cpu().numpy()
        for e in range(sh.E):
            assert np.linalg.norm(got[e] - ref[key][e]) <= c.rel * np.linalg.norm(ref[key][e]) + 1e-30, (key, e)


@pytest.mark.parametrize("one_call", [True, False])
def test_gate_products_of_tail_tiles(one_call):
    """K > 1, experts of a few rows up to 128: the products <dy, o> that the gate's gradient is made of come from pairs of waves."""
    sh = SH(T=300, d=512, E=24, K=4, F=512, sigma=0.05, zipf_s=0.8, seed=79)
    c = Case(sh, backward=True, scale_w=5.0)
    n = c.np
    fwd = sparse.forward(n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], n["bias"])
    ref = sparse.backward(n["dy"], n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], fwd, want_dbias=True)
    w = (c.t["Wg"], c.t["Wu"], c.t["Wd"])
    buf = r3.LayerBuffers(c.D, backward=True, gathered_copy=False)
    dbias = torch.zeros(sh.E, dtype=torch.float32, device="cuda")
    (r3.forward_one_call if one_call else r3.forward)(buf, c.t["x"], c.t["Wr"], c.t["idx"], *w, bias=c.t["bias"])
    r3.backward(buf, c.t["dy"], c.t["x"], c.t["Wr"], c.t["idx"], *w, dbias=dbias)
    torch.cuda.synchronize()
    sig_w, sig_b = router_gradient_sigma(n["x"], n["dy"], c.idx, fwd, sh.E)
    assert_close(buf.dW_r.cpu().numpy(), ref["dWr"], "dW_r", c.rel, sig_w)
    assert_close(dbias.cpu().numpy(), ref["dbias"], "dbias", c.rel, sig_b)
    assert_close(host(buf.dx), ref["dx"], "dx", c.rel)


def test_masked_lanes_of_sources_past_two_gigabytes():
    """Width 1032: the last window of a reduction has 8 live values, the other lanes fetch nothing, also where more than
    2 GB of the source are left: NaN in rows 2 GB on stay where they are."""
    T, d, E, F = 1 << 20, 1032, 64, 8
    D = r3.desc(T, d, E, 1, F)
    bad = (1 << 31) // (2 * d) - 1                       # NaN from the row that 2 GB from row 0 lie in
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.zeros(T, d, dtype=torch.bfloat16, device="cuda")
    x[:4096] = torch.randn(4096, d, generator=g, device="cuda")
    x[bad:] = float("nan")
    # router: one id per token (gate 1), logits kept
    Wr = torch.randn(d, E, generator=g, device="cuda").bfloat16()
    idx = torch.zeros(T, 1, dtype=torch.uint8, device="cuda")
    gates = torch.empty(T, 1, dtype=torch.float32, device="cuda")
    logits = torch.empty(T, E, dtype=torch.float32, device="cuda")
    r3.replay_gate(D, x, Wr, idx, gates, logits_out=logits, ws=r3.workspace(D, r3.OP_REPLAY_GATE))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(logits[:4096]).all()) and bool(torch.isnan(logits[bad:]).all())
    assert torch.allclose(logits[:4096].double(), x[:4096].double() @ Wr.double(), rtol=1e-4, atol=1e-3)
    del logits
    # expert network on rows that are there already, all of them of expert 0
    offsets = torch.full((E + 1,), T, dtype=torch.int32, device="cuda")
    offsets[0] = 0
    Wg, Wu = (0.05 * torch.randn(E, d, F, generator=g, device="cuda").bfloat16() for _ in range(2))
    Wd = torch.randn(E, F, d, generator=g, device="cuda").bfloat16()
    Yp, H = torch.empty(T, d, dtype=torch.bfloat16, device="cuda"), torch.empty(T, F, dtype=torch.bfloat16, device="cuda")
    r3.grouped_ffn(D, x, offsets, Wg, Wu, Wd, Yp, H, ws=r3.workspace(D, r3.OP_GROUPED_FFN))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(H[:4096]).all()) and bool(torch.isnan(H[bad:]).all())
    a, b = x[:4096].double() @ Wg[0].double(), x[:4096].double() @ Wu[0].double()
    want = a * torch.sigmoid(a) * b
    assert float((H[:4096].double() - want).norm() / want.norm()) < 4e-3      # (one rounding to bf16: 2^-9 at most)


def test_sigmoid_of_large_arguments():
    """FB = silu(A) at A = -80 .. -20, sums of two bf16 weights (exact in f32): next to none is rounded to bf16 on another side
    than the exact value.  An error of n ulp of f32 flips about n in 65536 (1 for expf and a division, 40 for the
    hardware's exponential of a rounded product)."""
    T, d, E, F = 512, 264, 1, 1032
    D = r3.desc(T, d, E, 1, F)
    g = torch.Generator(device="cuda").manual_seed(3)
    Wg = torch.zeros(E, d, F, device="cuda")
    Wg[:, :d // 2] = -20 - 50 * torch.rand(E, d // 2, F, generator=g, device="cuda")
    Wg[:, d // 2:] = -torch.rand(E, d // 2, F, generator=g, device="cuda")
    Wg = Wg.bfloat16()
    hi = torch.randint(0, d // 2, (T,), generator=g, device="cuda")
    lo = torch.randint(d // 2, d, (T,), generator=g, device="cuda")
    x = torch.zeros(T, d, device="cuda").scatter_(1, torch.stack([hi, lo], 1), 1.0).bfloat16()
    offsets = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    e = lambda n: torch.empty(T, n, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    Yp, H, FA, FB = e(d), e(F), e(F), e(F)
    r3.grouped_ffn(D, x, offsets, Wg, Wg, torch.zeros(E, F, d, device="cuda").bfloat16(), Yp, H, FA, FB,
                   ws=r3.workspace(D, r3.OP_GROUPED_FFN))
    torch.cuda.synchronize()
    a = Wg[0].double()[hi] + Wg[0].double()[lo]
    want = (a * torch.sigmoid(a)).bfloat16()
    flips = int((FB != want).sum())
    assert flips <= 4 * T * F / 65536, flips


@pytest.mark.parametrize("d,F", [(264, 136), (1000, 72), (256, 256)])     # (whole tiles beside the guarded ones)
def test_nonfinite_values_stay_where_they_belong(d, F):
    """NaN or infinity in the last value of a token, of its dy, or of one expert's weights: the tokens and experts that do not
    meet it come out finite, though masked lanes and dead rows lie beside it."""
    T, E, K = 700, 12, 3
    sh = SH(T=T, d=d, E=E, K=K, F=F, sigma=0.02, seed=77)
    c = Case(sh, backward=True, scale_w=5.0)
    idx = torch.from_numpy(c.idx).long().cuda()
    t0, e0 = 333, int(c.idx[333, 1])

    def run(**bad):
        t = {k: v.clone() if v is not None else None for k, v in c.t.items()}
        for k, (at, value) in bad.items():
            t[k][at] = value
        w = (t["Wg"], t["Wu"], t["Wd"])
        buf = r3.LayerBuffers(c.D, backward=True, gathered_copy=False)
        r3.forward_one_call(buf, t["x"], t["Wr"], t["idx"], *w, bias=t["bias"])
        r3.backward(buf, t["dy"], t["x"], t["Wr"], t["idx"], *w)
        torch.cuda.synchronize()
        return buf

    tokens = torch.arange(T, device="cuda")
    finite = lambda v: bool(torch.isfinite(v).all())    # noqa: E731
    other_experts = torch.ones(E, dtype=torch.bool, device="cuda")
    other_experts[idx[t0]] = False
    b = run(x=((t0, d - 1), float("nan")))
    assert not finite(b.y[t0]) and finite(b.y[tokens != t0]) and finite(b.dx[tokens != t0])
    assert all(finite(g[other_experts]) for g in (b.dW_gate, b.dW_up, b.dW_down))
    b = run(dy=((t0, d - 1), float("inf")))
    assert finite(b.y) and not finite(b.dx[t0]) and finite(b.dx[tokens != t0])
    assert all(finite(g[other_experts]) for g in (b.dW_gate, b.dW_up, b.dW_down))
    apart = (idx != e0).all(1)
    others = torch.arange(E, device="cuda") != e0
    for k, at in (("Wg", (e0, d - 1, F - 1)), ("Wu", (e0, 0, 0)), ("Wd", (e0, F - 1, d - 1)), ("Wd", (e0, 0, 0))):
        b = run(**{k: (at, float("nan"))})
        assert finite(b.y[apart]) and finite(b.dx[apart]) and not finite(b.y), k
        # (the tokens that met it carry it, through their gate's gradient, to their other experts' dz, not to their weights)
        assert all(finite(g[others]) for g in (b.dW_gate, b.dW_up, b.dW_down)), k


@pytest.mark.parametrize("one_call", [True, False])
@pytest.mark.parametrize("d,F", [(512, 512), (520, 392)])     # whole tiles; guarded ones
def test_gate_gradients_do_not_depend_on_the_batch(d, F, one_call):
    """A row's dz is the same bits whether its expert's rows make a tail tile or a full one: tokens without an upstream gradient
    behind the others lift every expert past 128 rows and leave dbias as it is."""
    few, many = 800, 2400
    sh = SH(T=many, d=d, E=64, K=8, F=F, sigma=0.02, seed=80)
    c = Case(sh, backward=True, scale_w=5.0)
    c.t["dy"][few:] = 0.0
    w, got = (c.t["Wg"], c.t["Wu"], c.t["Wd"]), []
    for T in (few, many):
        x, dy, idx = (c.t[k][:T].contiguous() for k in ("x", "dy", "idx"))
        buf = r3.LayerBuffers(r3.desc(T, d, sh.E, sh.K, F), backward=True, gathered_copy=False)
        dbias = torch.zeros(sh.E, dtype=torch.float32, device="cuda")
        (r3.forward_one_call if one_call else r3.forward)(buf, x, c.t["Wr"], idx, *w)
        r3.backward(buf, dy, x, c.t["Wr"], idx, *w, dbias=dbias)
        torch.cuda.synchronize()
        got.append((dbias, buf.dx[:few].clone(), buf.counts.tolist()))
    assert np.median(got[0][2]) <= 128 < min(got[1][2])
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("T,d,F", [(500, 392, 592), (8200, 40, 776)])     # H left in the caches; 102 MB of it streamed
def test_forward_without_saved_tensors(T, d, F):
    """Whether the forward saves for a backward does not change a bit of y."""
    sh = SH(T=T, d=d, E=16, K=8, F=F, sigma=0.02, seed=81)
    c = Case(sh, scale_w=5.0)
    y = []
    for backward in (False, True):
        buf = r3.LayerBuffers(c.D, backward=backward, gathered_copy=False)
        buf.H.fill_(7.0)
        r3.forward_one_call(buf, c.t["x"], c.t["Wr"], c.t["idx"], c.t["Wg"], c.t["Wu"], c.t["Wd"])
        torch.cuda.synchronize()
        y.append((buf.H, buf.y))
    assert torch.equal(y[0][0], y[1][0]) and torch.equal(y[0][1], y[1][1])
    n = c.np
    fwd = sparse.forward(n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], n["bias"])
    assert_close(host(y[0][1]), fwd["y"], "y", c.rel)
