"""The row kernels (combine; dx with the router's last step in its grid) where a block holds one, two, four or eight tokens and the last
one is not full, for every K they are compiled for and one they are not: against the same sums in float64 from the rows that the layer left."""
import numpy as np
import pytest
import torch

from oracle import sparse
from paper_2510_11370_amd import r3, synth
from util import Case, assert_close, dx_64, host

pytestmark = pytest.mark.gpu
SH = synth.LayerShape


@pytest.mark.parametrize("K", [1, 2, 3, 4, 6, 8])
@pytest.mark.parametrize("d,T", [(8, 8193), (264, 8195), (512, 4097), (1000, 2049), (2056, 1025), (1000, 37)])   # 1, 33, 64, 125, 257 vectors; too few tokens to share a block
def test_combine_and_dx_rows(d, T, K):
    for act, idx_E in (("bf16", 16), ("bf16", 264), ("f32", 16)):
        sh = SH(T=T, d=d, E=idx_E, K=K, F=8, act=act, sigma=0.02, seed=151)
        c = Case(sh, backward=True, scale_w=5.0)
        buf = r3.LayerBuffers(c.D, backward=True, gathered_copy=False)
        w = (c.t["Wg"], c.t["Wu"], c.t["Wd"])
        r3.forward(buf, c.t["x"], c.t["Wr"], c.t["idx"], *w, bias=c.t["bias"])
        r3.backward(buf, c.t["dy"], c.t["x"], c.t["Wr"], c.t["idx"], *w)
        torch.cuda.synchronize()
        rows = buf.inv_perm.long().view(T, K)
        want = (buf.gates.double()[:, :, None] * buf.Yp.double()[rows]).sum(1)
        # one rounding to the result's type, and K f32 additions
        rel = 2.0 ** -8 if act == "bf16" else 1e-6
        assert ((buf.y.double() - want).abs() <= rel * want.abs() + 1e-6 * want.abs().max()).all()
        # dA and dB, dXp and dx are rounded to the result's type, as are the rows that the reference's dz comes from; f32 sums of up to 2056 terms
        rel = 4 * 2.0 ** -9 if act == "bf16" else 1e-5
        assert ((buf.dx.double() - dx_64(c, buf, c.t["dy"])).abs() <= rel * dx_64(c, buf, c.t["dy"], scale=True)).all()


@pytest.mark.parametrize("sh", [
    SH(T=4100, d=256, E=8, K=2, F=264, sigma=0.02, seed=152),                   # 32 lanes a token, the last block half full
    SH(T=2051, d=520, E=300, K=4, F=72, sigma=0.02, seed=153),                  # 128 lanes, two-byte record
    SH(T=2050, d=1000, E=16, K=6, F=40, sigma=0.02, zipf_s=1.0, seed=154),
    SH(T=1030, d=2048, E=24, K=3, F=40, sigma=0.02, seed=155),                  # K that nothing is compiled for
    SH(T=301, d=68, E=40, K=9, F=36, act="f32", sigma=0.05, seed=156),          # f32, the gate's backward beside dH: 4 + 4 + 1 rows a token
    SH(T=38, d=516, E=300, K=33, F=36, act="f32", sigma=0.05, seed=157),        # two-byte record, two rounds of a wave's lanes along d
], ids=lambda s: "T%d_d%d_E%d_K%d" % (s.T, s.d, s.E, s.K))
def test_dx_with_the_routers_last_step(sh):
    c = Case(sh, backward=True, scale_w=5.0)
    n = c.np
    fwd = sparse.forward(n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], n["bias"])
    ref = sparse.backward(n["dy"], n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], fwd, want_dbias=True)
    w = (c.t["Wg"], c.t["Wu"], c.t["Wd"])
    buf = r3.LayerBuffers(c.D, backward=True, gathered_copy=False)
    dbias = torch.zeros(sh.E, dtype=torch.float32, device="cuda")
    r3.forward_one_call(buf, c.t["x"], c.t["Wr"], c.t["idx"], *w, bias=c.t["bias"])
    r3.backward(buf, c.t["dy"], c.t["x"], c.t["Wr"], c.t["idx"], *w, dbias=dbias)
    torch.cuda.synchronize()
    assert_close(host(buf.dx), ref["dx"], "dx", c.rel)
    for got, want in ((buf.dW_r.cpu().numpy(), ref["dWr"]), (dbias.cpu().numpy(), ref["dbias"])):
        assert np.linalg.norm(got - want) <= c.rel * np.linalg.norm(want)
