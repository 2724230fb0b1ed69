"""The f32-arithmetic tile kernels (f32 layers, and bf16 widths the bf16 matrix kernels do not take) at the edges of
their tiles: 32 x 32, 64 x 64 and 128 x 128 outputs, 32 k per step, four elements per load where the widths allow it.  Forward in
one call and backward, against the CPU oracle, with the bars of tests/util.py."""
import numpy as np
import pytest
import torch

from oracle import sparse
from paper_2510_11370_amd import r3, synth
from util import Case, assert_close, assert_gates_close, host, router_gradient_sigma

pytestmark = pytest.mark.gpu
SH = synth.LayerShape


@pytest.mark.parametrize("sh", [
    SH(T=1, d=33, E=3, K=1, F=31, act="f32", seed=61),                   # one row, one-element loads
    SH(T=65, d=64, E=2, K=1, F=128, act="f32", sigma=0.05, seed=62),     # whole tiles, one row over a tile
    SH(T=129, d=132, E=70, K=3, F=60, act="f32", sigma=0.05, seed=63),   # more experts than lanes, four elements over a tile
    SH(T=257, d=51, E=9, K=4, F=66, act="bf16", sigma=0.05, seed=64),    # bf16 widths no vector load fits
    SH(T=3, d=4, E=5, K=2, F=4, act="f32", seed=66),                      # one 16-byte piece a row, experts without rows
    SH(T=96, d=36, E=2, K=1, F=100, act="f32", sigma=0.05, seed=67),      # 32 x 32 tiles, a k-tile's second piece alone
    SH(T=1030, d=68, E=3, K=2, F=640, act="f32", sigma=0.05, seed=68),    # 64 x 64 tiles forward (10 to a row), 32 x 32 backward
    SH(T=700, d=516, E=4, K=3, F=1028, act="f32", sigma=0.05, zipf_s=1.0, seed=69),   # 64 x 64 tiles all through, four over a tile
    SH(T=2050, d=1028, E=10, K=4, F=1028, act="f32", sigma=0.05, zipf_s=0.7, seed=65),   # the 128 x 128 tiles, ragged on every side
], ids=lambda s: "T%d_d%d_F%d_E%d_K%d_%s" % (s.T, s.d, s.F, s.E, s.K, s.act))
def test_layer_at_tile_edges(sh):
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
    assert int(buf.status.item()) == 0
    assert_gates_close(buf.gates.cpu().numpy(), fwd["g"])
    assert_close(host(buf.y), fwd["y"], "y", c.rel)
    assert_close(host(buf.dx), ref["dx"], "dx", c.rel)
    sig_w, sig_b = (None, None) if sh.act == "f32" else router_gradient_sigma(n["x"], n["dy"], c.idx, fwd, sh.E)
    if sh.K > 1:      # (with one expert per token the gate is the constant 1 and the router gradient exactly 0)
        assert_close(buf.dW_r.cpu().numpy(), ref["dWr"], "dW_r", c.rel, sig_w)
        assert_close(dbias.cpu().numpy(), ref["dbias"], "dbias", c.rel, sig_b)
    else:
        assert not buf.dW_r.any() and not dbias.any()
    for got, key in ((buf.dW_gate, "dWg"), (buf.dW_up, "dWu"), (buf.dW_down, "dWd")):
        got = got.cpu().numpy()
        for e in range(sh.E):
            assert np.linalg.norm(got[e] - ref[key][e]) <= c.rel * np.linalg.norm(ref[key][e]) + 1e-30, (key, e)
