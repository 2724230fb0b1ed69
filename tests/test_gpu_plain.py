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
    SH(T=1030, d=68, E=3, K=2, F=640, act="f32", sigma=0.05, seed=68),    # 64 x 64 tiles in the SwiGLU (20 to a row), 32 x 32 in the rest
    SH(T=700, d=516, E=4, K=3, F=1028, act="f32", sigma=0.05, zipf_s=1.0, seed=69),   # 64 x 64 tiles but for outputs of width d, four over a tile
    SH(T=2050, d=1028, E=10, K=4, F=1028, act="f32", sigma=0.05, zipf_s=0.7, seed=65),   # 64 x 64 tiles all through, ragged on every side
    SH(T=2050, d=1028, E=10, K=4, F=1028, act="bf16", sigma=0.05, zipf_s=0.7, seed=84),  # the 128 x 128 tiles, ragged on every side
    SH(T=257, d=52, E=9, K=4, F=68, act="bf16", sigma=0.05, seed=85),     # bf16 in vector loads, 64 x 64 tiles
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


@pytest.mark.parametrize("sh", [
    SH(T=70, d=36, E=300, K=3, F=44, act="f32", sigma=0.05, seed=71),             # two-byte record
    SH(T=330, d=132, E=9, K=2, F=68, act="f32", sigma=0.05, zipf_s=0.8, seed=72),  # one-byte record, tiles cut on every side
], ids=lambda s: "T%d_d%d_F%d_E%d_K%d" % (s.T, s.d, s.F, s.E, s.K))
def test_shared_launches_of_the_f32_backward(sh):
    """A token-major record, accumulated gradients, and tokens through perm or expert-sorted, after the one-call forward: the
    kernels that share a launch there against the oracle, and against each other bit for bit."""
    c = Case(sh, backward=True, scale_w=5.0)
    n, L = c.np, 3
    fwd = sparse.forward(n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], n["bias"])
    ref = sparse.backward(n["dy"], n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], fwd, want_dbias=True)
    D = r3.desc(sh.T, sh.d, sh.E, sh.K, sh.F, act="f32", idx_token_stride=L * sh.K)
    record = torch.zeros(sh.T, L, sh.K, dtype=torch.uint8 if sh.E <= 256 else torch.uint16, device="cuda")
    record[:, 1] = c.t["idx"]
    idx, w = record[:, 1], (c.t["Wg"], c.t["Wu"], c.t["Wd"])
    buf = r3.LayerBuffers(D, backward=True, gathered_copy=False)
    r3.forward_one_call(buf, c.t["x"], c.t["Wr"], idx, *w, bias=c.t["bias"])
    perm = torch.from_numpy(fwd["perm"].astype(np.int64)).cuda()
    results = []
    for Xp in (None, c.t["x"][perm // sh.K].contiguous()):
        dbias = torch.zeros(sh.E, dtype=torch.float32, device="cuda")
        for accumulate in (False, True):
            r3.moe_backward(r3.gated_desc(D), c.t["dy"], c.t["x"], c.t["Wr"], idx, buf.gates, buf.inv_perm, buf.perm, buf.offsets,
                            Xp, buf.A, buf.B, buf.H, buf.Yp, *w, buf.dx, buf.dW_r, buf.dW_gate, buf.dW_up, buf.dW_down,
                            buf.ws_bwd, dbias=dbias, accumulate=accumulate)
            torch.cuda.synchronize()
            times = 2.0 if accumulate else 1.0
            assert_close(host(buf.dx), ref["dx"], "dx", c.rel)
            assert_close(buf.dW_r.cpu().numpy(), times * ref["dWr"], "dW_r", c.rel)
            assert_close(dbias.cpu().numpy(), times * ref["dbias"], "dbias", c.rel)
            for got, key in ((buf.dW_gate, "dWg"), (buf.dW_up, "dWu"), (buf.dW_down, "dWd")):
                got = got.cpu().numpy()
                for e in range(sh.E):
                    want = times * ref[key][e]
                    assert np.linalg.norm(got[e] - want) <= c.rel * np.linalg.norm(want) + 1e-30, (key, e)
        results.append([t.clone() for t in (buf.dx, buf.dW_r, buf.dW_gate, buf.dW_up, buf.dW_down, dbias)])
    for a, b in zip(*results):
        assert torch.equal(a, b)


def chains_of_1024(v):
    """The float32 sum of an expert's dz as the library orders it: 1024 chains of every 1024th row, four rows to an addition, a
    butterfly over each 64 chains, the sixteen results one after the other."""
    v = np.concatenate([v, np.zeros(-len(v) % 4096, np.float32)]).reshape(-1, 4, 1024)
    chain = np.zeros(1024, np.float32)
    for a in v:
        chain = chain + ((a[0] + a[1]) + (a[2] + a[3]))
    w = chain.reshape(16, 64)
    for o in (32, 16, 8, 4, 2, 1):
        w = w + w[:, np.arange(64) ^ o]
    total = np.float32(0.0)
    for s in w[:, 0]:
        total = total + s
    return total


@pytest.mark.parametrize("one_call", [True, False])
def test_router_bias_of_long_segments(one_call):
    """dbias of an f32 layer, an expert of 70001 rows among them, is the sum of 1024 chains per expert (fewer chains round more),
    whatever launch makes it.  The experts' weights do not touch the upper half of x and W_r is the unit matrix there, so that
    dx shows every dz as it is."""
    T, E, d, F = 70001, 5, 16, 8
    g = torch.Generator().manual_seed(91)
    x, dy = torch.randn(T, d, generator=g), torch.randn(T, d, generator=g)
    Wr = torch.zeros(d, E)
    Wr[8:8 + E] = torch.eye(E)
    Wg, Wu, Wd = (torch.randn(E, a, b, generator=g) for a, b in ((d, F), (d, F), (F, d)))
    Wg[:, 8:] = 0.0
    Wu[:, 8:] = 0.0
    idx = torch.stack([torch.zeros(T, dtype=torch.int64), torch.randint(1, E, (T,), generator=g)], 1).to(torch.uint8)
    x, dy, Wr, Wg, Wu, Wd, idx = (t.cuda().contiguous() for t in (x, dy, Wr, Wg, Wu, Wd, idx))
    buf = r3.LayerBuffers(r3.desc(T, d, E, 2, F, act="f32"), backward=True, gathered_copy=False)
    dbias = torch.zeros(E, dtype=torch.float32, device="cuda")
    (r3.forward_one_call if one_call else r3.forward)(buf, x, Wr, idx, Wg, Wu, Wd)
    r3.backward(buf, dy, x, Wr, idx, Wg, Wu, Wd, dbias=dbias)
    torch.cuda.synchronize()
    dz, chosen = buf.dx[:, 8:8 + E].cpu().numpy(), idx.cpu().numpy()
    for e in range(E):
        rows = dz[(chosen == e).any(1), e]
        assert len(rows) > 16000 and (rows != 0).mean() > 0.9
        assert dbias[e].item() == chains_of_1024(rows), e
