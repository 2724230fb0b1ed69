"""bf16 backward: launches that share their work-groups (dH with dW_down, dXp with dW_gate and dW_up) and those that do not, on both sides of
the rule, against the CPU oracle; a work-group then has tiles of both sorts, of one, or none."""
import numpy as np
import pytest
import torch

from oracle import sparse
from paper_2510_11370_amd import r3, synth
from util import Case, assert_close, host, router_gradient_sigma

pytestmark = pytest.mark.gpu
SH = synth.LayerShape


@pytest.mark.parametrize("copy", [False, True], ids=["gathered", "Xp"])
@pytest.mark.parametrize("sh", [
    SH(T=1, d=256, E=1, K=1, F=256, seed=141),                                   # a tile or two in each launch
    SH(T=600, d=256, E=6, K=4, F=256, sigma=0.02, zipf_s=0.9, seed=142),         # both shared, fewer tiles than work-groups
    SH(T=601, d=264, E=5, K=3, F=392, sigma=0.02, zipf_s=1.2, seed=143),         # both shared, ragged widths
    SH(T=2047, d=512, E=20, K=16, F=256, sigma=0.02, zipf_s=0.5, seed=144),      # just under 128 F slots: shared
    SH(T=2048, d=512, E=20, K=16, F=256, sigma=0.02, zipf_s=0.5, seed=145),      # reductions may be cut: each its own launch
    SH(T=2500, d=1000, E=16, K=4, F=704, sigma=0.02, zipf_s=1.0, seed=146),      # more tiles than work-groups in both, ragged
    SH(T=900, d=128, E=100, K=6, F=264, sigma=0.02, zipf_s=1.0, seed=147),       # experts ranked by two waves, many of a size
    SH(T=900, d=128, E=1100, K=2, F=264, sigma=0.02, zipf_s=1.0, seed=148),      # more experts than threads rank
], ids=lambda s: "T%d_d%d_F%d_E%d" % (s.T, s.d, s.F, s.E))
def test_gradients(sh, copy):
    c = Case(sh, backward=True, scale_w=5.0)
    n = c.np
    fwd = sparse.forward(n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], n["bias"])
    ref = sparse.backward(n["dy"], n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], fwd)
    sig, _ = router_gradient_sigma(n["x"], n["dy"], c.idx, fwd, sh.E)
    w = (c.t["Wg"], c.t["Wu"], c.t["Wd"])
    buf = r3.LayerBuffers(c.D, backward=True, gathered_copy=False)
    r3.forward_one_call(buf, c.t["x"], c.t["Wr"], c.t["idx"], *w, bias=c.t["bias"])
    Xp = c.t["x"][buf.perm.long() // sh.K].contiguous() if copy else None
    first = None
    for accumulate in (False, True):
        r3.moe_backward(r3.gated_desc(c.D), c.t["dy"], c.t["x"], c.t["Wr"], c.t["idx"], buf.gates, buf.inv_perm, buf.perm, buf.offsets, Xp,
                        buf.A, buf.B, buf.H, buf.Yp, *w, buf.dx, buf.dW_r, buf.dW_gate, buf.dW_up, buf.dW_down, buf.ws_bwd,
                        accumulate=accumulate)
        torch.cuda.synchronize()
        grads = [buf.dW_gate, buf.dW_up, buf.dW_down]
        if first is None:
            first = [g.clone() for g in grads] + [buf.dx.clone()]
            assert_close(host(buf.dx), ref["dx"], "dx", c.rel)
            if sh.K > 1:
                assert_close(buf.dW_r.cpu().numpy(), ref["dWr"], "dW_r", c.rel, sig)
            for got, key in zip(grads, ("dWg", "dWu", "dWd")):
                got = got.cpu().numpy()
                for e in range(sh.E):
                    assert np.linalg.norm(got[e] - ref[key][e]) <= c.rel * np.linalg.norm(ref[key][e]) + 1e-30, (key, e)
        else:   # whichever work-group ran what: the same sums, added to what was there
            assert torch.equal(first[3], buf.dx)
            for a, g in zip(first, grads):
                assert torch.equal(a + a, g)
