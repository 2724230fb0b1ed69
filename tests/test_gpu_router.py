"""The router kernels (logits, replay gate, agreement; their weight gradient) and the dispatch at the edges of their tiles and of the rule that picks
between them, against the CPU oracle: gates to 1e-5 (tests/util.py), logits to a float32 sum's error, status and agreement."""
import numpy as np
import pytest
import torch

from oracle import sparse
from paper_2510_11370_amd import r3, synth
from util import Case, assert_close, assert_gates_close, router_gradient_sigma

pytestmark = pytest.mark.gpu
SH = synth.LayerShape


@pytest.mark.parametrize("sh", [
    SH(T=1, d=8, E=8, K=8, F=8, seed=81),                            # one token, one piece of k
    SH(T=33, d=264, E=72, K=6, F=8, zipf_s=0.5, seed=82),            # a token, a piece of k and an expert over the tiles
    SH(T=64, d=1000, E=264, K=12, F=8, seed=83),                     # four expert groups; K > 8: agreement by its own launch
    SH(T=130, d=512, E=512, K=8, F=8, seed=84),                      # the most experts of the bf16 kernel
    SH(T=70, d=256, E=640, K=4, F=8, seed=85),                       # beyond it
    SH(T=8192, d=64, E=128, K=8, F=8, seed=86), SH(T=8193, d=64, E=128, K=8, F=8, seed=87),       # 32 | 64 tokens
    SH(T=32768, d=64, E=128, K=8, F=8, seed=88), SH(T=32769, d=64, E=128, K=8, F=8, seed=89),     # 64 | 128 tokens
    SH(T=17, d=50, E=60, K=5, F=8, seed=90),                         # bf16 in f32 arithmetic
    SH(T=49, d=132, E=9, K=3, F=8, act="f32", seed=91), SH(T=16, d=129, E=128, K=8, F=8, act="f32", zipf_s=0.7, seed=92),
    SH(T=40, d=33, E=130, K=2, F=8, act="f32", seed=93),             # more experts than the f32 kernel holds
], ids=lambda s: "T%d_d%d_E%d_K%d_%s" % (s.T, s.d, s.E, s.K, s.act))
def test_router_at_tile_edges(sh):
    c = Case(sh, backward=False)
    gates = torch.empty(sh.T, sh.K, dtype=torch.float32, device="cuda")
    logits = torch.full((sh.T + 1, sh.E), 7.0, dtype=torch.float32, device="cuda")     # a row to spare: nothing past the end
    agree = torch.zeros(2, dtype=torch.int64, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = r3.workspace(c.D, r3.OP_REPLAY_GATE)
    r3.replay_gate(c.D, c.t["x"], c.t["Wr"], c.t["idx"], gates, bias=c.t["bias"], logits_out=logits, agree_out=agree,
                   status=status, ws=ws)
    torch.cuda.synchronize()
    lg = logits.cpu().numpy()
    assert (lg[-1] == 7.0).all() and int(status.item()) == 0
    lg = lg[:-1]
    assert np.abs(lg - c.s).max() <= 2e-5 * max(1.0, np.abs(c.s).max())
    assert_gates_close(gates.cpu().numpy(), sparse.replay_gate(c.s, c.idx))
    # the counts are of the kernel's own logits: exact against the oracle's selection on those
    own = sparse.topk_mask(lg, sh.K)
    assert tuple(agree.tolist()) == tuple(int(v) for v in sparse.agreement(own, c.idx))
    # logits kept on chip: the same gates and counts
    gates2 = torch.empty_like(gates)
    r3.replay_gate(c.D, c.t["x"], c.t["Wr"], c.t["idx"], gates2, bias=c.t["bias"], agree_out=agree, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(gates, gates2)
    assert tuple(agree.tolist()) == tuple(2 * int(v) for v in sparse.agreement(own, c.idx))


@pytest.mark.parametrize("E,d", [(64, 264), (128, 512), (128, 264), (256, 328), (384, 136), (512, 256)])
def test_logits_do_not_depend_on_the_batch(E, d):
    """A token's logits and gates are the same bits whatever the number of tokens in the call: micro-batches replay as
    the whole batch does.  32 | 64 | (E = 128) 128 tokens per work-group."""
    T, K = 33000, 4
    g = torch.Generator(device="cuda").manual_seed(E + d)
    x = torch.randn(T, d, generator=g, device="cuda").bfloat16()
    Wr = torch.randn(d, E, generator=g, device="cuda").bfloat16()
    idx = (torch.randint(0, E // K, (T, K), generator=g, device="cuda") + E // K * torch.arange(K, device="cuda")).to(
        torch.uint8 if E <= 256 else torch.int16)
    got = []
    for n in (T, 32768, 9000, 8192, 33):
        D = r3.desc(n, d, E, K, 8)
        lg, gates = (torch.empty(n, w, dtype=torch.float32, device="cuda") for w in (E, K))
        r3.replay_gate(D, x[:n], Wr, idx[:n], gates, logits_out=lg, ws=r3.workspace(D, r3.OP_REPLAY_GATE))
        got.append((n, lg, gates))
    torch.cuda.synchronize()
    for n, lg, gates in got[1:]:
        assert torch.equal(lg, got[0][1][:n]) and torch.equal(gates, got[0][2][:n]), n


@pytest.mark.parametrize("T,E,d,act", [
    (200, 128, 256, "bf16"), (9000, 64, 72, "bf16"), (200, 384, 256, "bf16"),      # a work-group of 32 | 64 tokens, all experts
    (33000, 128, 64, "bf16"),                                                      # the kernel for many tokens
    (200, 16, 48, "f32"), (200, 60, 50, "bf16"),                                   # f32 arithmetic in one launch
    (200, 640, 256, "bf16"), (200, 130, 33, "f32"),                                # logits and gates in a launch each
])
def test_every_gate_kernel_flags_bad_records_and_nonfinite_logits(T, E, d, act):
    """An id past the last expert, in the last token, and a non-finite logit raise their bits, and only their own token's
    gates change."""
    K = 4
    D = r3.desc(T, d, E, K, 256, act)
    g = torch.Generator(device="cuda").manual_seed(T + E)
    a = r3.act_dtype(D)
    x = torch.randn(T, d, generator=g, device="cuda").to(a)
    Wr = (torch.randn(d, E, generator=g, device="cuda") * d ** -0.5).to(a)
    idx = torch.randint(0, E // K, (T, K), generator=g, device="cuda") + E // K * torch.arange(K, device="cuda")
    ids = lambda t: t.to(torch.uint8) if E <= 256 else t.to(torch.int16)   # noqa: E731

    def run(xx, rec):
        gates = torch.empty(T, K, dtype=torch.float32, device="cuda")
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        agree = torch.zeros(2, dtype=torch.int64, device="cuda")
        r3.replay_gate(D, xx, Wr, ids(rec), gates, status=status, agree_out=agree, ws=r3.workspace(D, r3.OP_REPLAY_GATE))
        torch.cuda.synchronize()
        return int(status.item()), gates

    st, clean = run(x, idx)
    assert st == 0 and torch.allclose(clean.sum(1), torch.ones(T, device="cuda"), atol=1e-5)
    bad = idx.clone()
    bad[T - 1, 1] = 255 if E <= 256 else 700
    st, got = run(x, bad)
    assert st == r3.DATA_IDX_RANGE and torch.equal(got[:-1], clean[:-1])
    xn = x.clone()
    xn[T - 2, d - 1] = float("inf")
    st, got = run(xn, idx)
    assert st == r3.DATA_NONFINITE
    keep = torch.arange(T, device="cuda") != T - 2
    assert torch.equal(got[keep], clean[keep])
    assert run(xn, bad)[0] == r3.DATA_NONFINITE | r3.DATA_IDX_RANGE


@pytest.mark.parametrize("T,E,K", [
    (700, 40, 3), (700, 250, 8), (2730, 100, 6),        # counted in one launch; ids that share lanes with their token and not
    (2731, 100, 6), (9000, 200, 2), (4000, 700, 8),     # counted by chunk first
    (900, 2000, 6),                                     # three launches
])
@pytest.mark.parametrize("token_major", [False, True])
def test_dispatch_flags_bad_records(T, E, K, token_major):
    """An id past the last expert (clamped) and a duplicate, late in the record: the bits, and the dispatch of what is left."""
    rng = np.random.default_rng(T + E)
    w = E // K
    idx = (rng.integers(0, w - 1, (T, K)) + w * np.arange(K)).astype(np.int32)     # (the last expert is nobody's)
    D = r3.desc(T, 16, E, K, 16, idx_token_stride=3 * K if token_major else 0)
    npdt = np.uint8 if E <= 256 else np.uint16
    cases = [(idx, 0)]
    bad = idx.copy(); bad[T - 2, K - 1] = np.iinfo(npdt).max; cases.append((bad, r3.DATA_IDX_RANGE))   # noqa: E702
    dup = idx.copy(); dup[T - 1, K - 1] = dup[T - 1, 0]; cases.append((dup, r3.DATA_IDX_DUP))          # noqa: E702
    both = bad.copy(); both[T - 1] = dup[T - 1]; cases.append((both, r3.DATA_IDX_RANGE | r3.DATA_IDX_DUP))   # noqa: E702
    for ids, bits in cases:
        rec = np.zeros((T, 3 if token_major else 1, K), npdt)
        rec[:, -1 if token_major else 0] = ids
        rec = torch.from_numpy(rec.view(np.int16) if E > 256 else rec).cuda()
        rec = rec[:, -1] if token_major else rec
        out = [torch.full((n,), -1, dtype=torch.int32, device="cuda") for n in (E, E + 1, T * K, T * K)]
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        r3.permute(D, None, rec, *out, None, r3.workspace(D, r3.OP_PERMUTE), status)
        torch.cuda.synchronize()
        assert int(status.item()) == bits
        for got, want in zip(out, sparse.permute(np.minimum(ids, E - 1), E)):
            assert np.array_equal(got.cpu().numpy(), want)


def _slots(T, E, K, seed, skew):
    rng = np.random.default_rng(seed)
    p = rng.random((T, E)) - skew * np.log(np.arange(1, E + 1))
    return np.sort(np.argsort(-p, axis=1)[:, :K], axis=1).astype(np.int32)


@pytest.mark.parametrize("T,E,K,skew,token_major", [
    (1, 1, 1, 0.0, False), (16384, 8, 1, 0.0, False),           # one slot; the most one launch counts by itself
    (5462, 100, 3, 0.3, True), (2731, 256, 6, 0.0, False),      # the first sizes counted by chunk; ids that fit no vector
    (2049, 128, 8, 0.5, True), (129, 1024, 64, 0.0, False),     # a slot over a chunk; the most experts of these kernels
    (300, 1025, 4, 0.0, False),                                 # beyond them
    (70000, 16, 16, 0.0, False), (131072, 128, 8, 0.3, False),  # several steps per wave
])
def test_dispatch_at_chunk_edges(T, E, K, skew, token_major):
    idx = _slots(T, E, K, T + E, skew)
    counts, offsets, inv_perm, perm = sparse.permute(idx, E)
    L = 3 if token_major else 1
    D = r3.desc(T, 16, E, K, 16, idx_token_stride=L * K if token_major else 0)
    rec = np.zeros((T, L, K), np.uint8 if E <= 256 else np.uint16)
    rec[:, L // 2] = idx
    rec = torch.from_numpy(rec.view(np.int16) if E > 256 else rec).to("cuda")
    if E > 256:
        rec = rec.view(torch.uint16)
    out = [torch.full((n,), -1, dtype=torch.int32, device="cuda") for n in (E, E + 1, T * K, T * K)]
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    r3.permute(D, None, rec[:, L // 2], *out, None, r3.workspace(D, r3.OP_PERMUTE), status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    for got, want in zip(out, (counts, offsets, inv_perm, perm)):
        assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("T,d,E,K,act,perm", [
    (1, 8, 8, 1, "bf16", "own"), (4097, 264, 130, 16, "bf16", "own"), (300, 128, 128, 24, "bf16", "own"),   # tile and part edges
    (65, 136, 130, 17, "bf16", "own"), (200, 128, 136, 33, "bf16", "own"), (2200, 64, 260, 64, "bf16", "own"),   # entries in batches
    (129, 33, 9, 3, "f32", "own"),                                                                         # the f32 tiles
    # Xp given: no perm, or one that holds nothing
    (65, 136, 136, 6, "bf16", None), (65, 136, 136, 6, "bf16", "unfilled"), (700, 136, 300, 4, "bf16", None),
    (150, 36, 70, 5, "f32", None), (150, 36, 70, 5, "f32", "unfilled"), (222, 64, 260, 7, "f32", None),
])
@pytest.mark.parametrize("token_major", [False, True])
def test_router_gradient_at_tile_edges(T, d, E, K, act, perm, token_major):
    """dW_r and dbias through r3_moe_backward, overwritten and then added to: after the forward in one call, and after the
    forward step by step without a permutation."""
    sh = SH(T=T, d=d, E=E, K=K, F=256, act=act, sigma=0.05, seed=95)
    c = Case(sh, backward=True, scale_w=5.0)
    n = c.np
    fwd = sparse.forward(n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], n["bias"])
    ref = sparse.backward(n["dy"], n["x"], n["Wr"], c.idx, n["Wg"], n["Wu"], n["Wd"], fwd, want_dbias=True)
    D, idx = c.D, c.t["idx"]
    if token_major:      # the middle one of three layers
        D = r3.desc(T, d, E, K, 256, act, idx_token_stride=3 * K)
        ids = idx if E <= 256 else idx.view(torch.int16)
        rec = torch.zeros(T, 3, K, dtype=ids.dtype, device="cuda")
        rec[:, 1] = ids
        idx = (rec if E <= 256 else rec.view(torch.uint16))[:, 1]
    buf = r3.LayerBuffers(D, backward=True, gathered_copy=perm != "own")
    w = (c.t["Wg"], c.t["Wu"], c.t["Wd"])
    (r3.forward_one_call if perm == "own" else r3.forward)(buf, c.t["x"], c.t["Wr"], idx, *w, bias=c.t["bias"])
    buf.perm = buf.perm if perm == "own" else None if perm is None else torch.zeros_like(buf.perm)
    dbias = torch.full((E,), 3.0, dtype=torch.float32, device="cuda")
    for acc in (False, True):
        r3.backward(buf, c.t["dy"], c.t["x"], c.t["Wr"], idx, *w, dbias=dbias, accumulate=acc)
    torch.cuda.synchronize()
    if K == 1:
        assert not buf.dW_r.any() and not dbias.any()
        return
    sw, sb = (None, None) if act == "f32" else router_gradient_sigma(n["x"], n["dy"], c.idx, fwd, E)
    assert_close(buf.dW_r.cpu().numpy() / 2, ref["dWr"], "dW_r", c.rel, sw)
    assert_close(dbias.cpu().numpy() / 2, ref["dbias"], "dbias", c.rel, sb)


def test_router_gradient_of_many_experts_a_token_stays_on_the_bf16_tiles():
    """From 16 to 17 experts a token the router's weight gradient costs a few percent more, not fifteen times as much
    (which the f32 tiles take: 3 is far from both)."""
    T, d, E, F, us = 8192, 1024, 128, 256, {}
    for K in (16, 17, 32):
        D = r3.desc(T, d, E, K, F)
        g = torch.Generator(device="cuda").manual_seed(K)
        rnd = lambda *s: (0.05 * torch.randn(*s, generator=g, device="cuda")).bfloat16()  # noqa: E731
        x, dy, Wr, w = rnd(T, d), rnd(T, d), rnd(d, E), (rnd(E, d, F), rnd(E, d, F), rnd(E, F, d))
        idx = torch.rand(T, E, generator=g, device="cuda").topk(K, 1).indices.sort(1).values.to(torch.uint8)
        buf = r3.LayerBuffers(D, backward=True, gathered_copy=False)
        r3.forward_one_call(buf, x, Wr, idx, *w)
        r3.backward(buf, dy, x, Wr, idx, *w)
        torch.cuda.synchronize()
        r3.profile_enable(True)
        for _ in range(5):
            r3.backward(buf, dy, x, Wr, idx, *w)
        torch.cuda.synchronize()
        ms, n = r3.profile_read()["router_wgrad"]
        r3.profile_enable(False)
        us[K] = 1e3 * ms / n
    assert us[17] < 3 * us[16] and us[32] < 3 * us[16], us


@pytest.mark.parametrize("T,E,K,pad", [(1, 1, 1, 0), (33, 5, 3, 0), (65, 33, 8, 3), (31, 100, 6, 4), (40, 257, 8, 0),
                                       (64, 384, 4, 0), (7, 385, 7, 1), (90, 512, 8, 0), (33, 513, 8, 0)])
def test_record_at_tile_edges(T, E, K, pad):
    """TopKMask for expert counts that fill no whole pieces: ties, NaNs and infinities included, rows `pad` floats apart."""
    rng = np.random.default_rng(E)
    lg = rng.integers(-3, 4, size=(T, E + pad)).astype(np.float32)
    lg[rng.random(lg.shape) < 0.05] = np.nan
    lg[rng.random(lg.shape) < 0.02] = -np.inf
    lg[0] = np.nan
    lg[:, E:] = 9.0                                    # beyond the row: never selected
    D = r3.desc(T, 16, E, K, 16)
    out = torch.zeros(T, K, dtype=torch.uint8 if E <= 256 else torch.int16, device="cuda")
    out = out if E <= 256 else out.view(torch.uint16)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    r3.record_topk(D, torch.from_numpy(lg).to("cuda"), out, status)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().astype(np.int32), sparse.topk_mask(np.ascontiguousarray(lg[:, :E]), K))
    assert int(status.item()) == r3.DATA_NONFINITE
