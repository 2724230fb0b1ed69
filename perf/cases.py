"""Performance cases of the replayed MoE layer: what users of this library have it do, from single small calls to the
largest training batches, through the public entry points of ``paper_2510_11370_amd.r3``.

Three kinds of case:

``layer``  one MoE layer as a training or recompute pass runs it: the record made from the rollout's logits
           (``record_topk``), the replayed forward (one call, or step by step) and, for training, the backward.
``cache``  the router-mask cache beside a paged KV cache: append the masks of a rollout, gather a packed batch.
``diag``   the training/inference discrepancy diagnostics: routing differences and the k3 / F(tau) estimates.

``listed()`` names the sizes, ``draw()`` gives further ones of the same ranges.  The 2048 x 768 x 128-expert, top-8 layer
is the one ``bench.py`` runs; the other widths are those of the tests or generic.
"""
import math

import numpy as np
import torch

from paper_2510_11370_amd import r3, synth

TAUS = [1.0, 1.5, 2.0, 4.0, 10.0]


def _layer(name, act, T, d, E, K, F, backward, zipf=0.0, sigma=0.01, calls="one", agree=False, dbias=False,
           token_major=False):
    return {"name": name, "kind": "layer", "act": act, "T": T, "d": d, "E": E, "K": K, "F": F, "backward": backward,
            "zipf": zipf, "sigma": sigma, "calls": calls, "agree": agree, "dbias": dbias, "token_major": token_major}


def listed():
    return [
        # the smallest use: a float32 layer of the unit-test size, where launches and host calls are the time
        _layer("train_f32_tiny", "f32", 256, 128, 8, 2, 256, True, sigma=0.05),
        # full-precision training of a small model (numerics studies against a bf16 run)
        _layer("train_f32_2k", "f32", 2048, 512, 16, 4, 1024, True, sigma=0.05),
        # recompute of a short continuation after a prefix-cache hit: 64 tokens meet every expert's weights
        _layer("fwd_64", "bf16", 64, 2048, 128, 8, 768, False),
        # recompute stage on one 4096-token micro-batch, forward only
        _layer("fwd_4k", "bf16", 4096, 2048, 128, 8, 768, False),
        # one layer of the 48-layer record + replay pass over 64 sequences x 2048 tokens, with agreement counts
        _layer("fwd_128k_agree", "bf16", 131072, 2048, 128, 8, 768, False, agree=True),
        # a small training micro-batch of odd length: the weights and their gradients are most of the traffic
        _layer("train_1k", "bf16", 1001, 2048, 128, 8, 768, True),
        # the ordinary training step
        _layer("train_16k", "bf16", 16384, 2048, 128, 8, 768, True),
        # the largest training step, with a router bias that makes the load Zipf-skewed
        _layer("train_64k_zipf", "bf16", 65536, 2048, 128, 8, 768, True, zipf=1.2),
        # widths that are no multiple of 256, 64 experts, top-6, odd token count
        _layer("train_ragged_3k", "bf16", 3001, 1000, 64, 6, 704, True, sigma=0.02),
        # more than 256 experts (uint16 record, kept token-major), forward call by call, the router bias trained too
        _layer("train_u16_6k", "bf16", 6000, 1024, 384, 4, 512, True, zipf=1.0, sigma=0.02, calls="steps", dbias=True,
               token_major=True),
        # masks of a whole 131072-token rollout stored and gathered again, 48 layers, pages of 16 tokens
        {"name": "mask_cache_128k", "kind": "cache", "L": 48, "T": 131072, "K": 8, "E": 128, "P": 16, "group": 4},
        # discrepancy report over a record pair of the same size and ten million sampled tokens
        {"name": "diagnostics_10m", "kind": "diag", "L": 48, "T": 131072, "K": 8, "E": 128, "n": 10_000_000,
         "token_major": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _ffn_flops(c):
    return (18.0 if c["backward"] else 6.0) * c["T"] * c["K"] * c["d"] * c["F"]


def _fit(c, flops):
    """Fewer tokens where the widths drawn would make the case dearer than the largest listed one of its sort."""
    most = flops * c["T"] / _ffn_flops(c)
    c["T"] = max(1, min(c["T"], int(most)))
    return c


def draw(rng):
    sort = rng.choice(["forward"] * 4 + ["train"] * 5 + ["ragged"] * 3 + ["f32"] * 3 + ["cache"] * 2 + ["diag"] * 2)
    if sort == "cache":
        return {"kind": "cache", "L": rng.choice([4, 24, 48, 61]), "T": _log(rng, 64, 131072 * 48 // 61),
                "K": rng.choice([2, 4, 6, 8]), "E": rng.choice([64, 128, 256, 384]), "P": rng.choice([8, 16, 64]),
                "group": rng.choice([1, 4, 8])}
    if sort == "diag":
        return {"kind": "diag", "L": rng.choice([4, 24, 48]), "T": _log(rng, 256, 131072), "K": rng.choice([2, 4, 6, 8]),
                "E": rng.choice([64, 128, 256, 384]), "n": _log(rng, 1000, 10_000_000), "token_major": rng.random() < 0.3}
    zipf = rng.choice([0.0, 0.0, round(rng.uniform(0.3, 1.3), 2)])
    sigma = rng.choice([0.01, 0.02, 0.05])
    calls = rng.choice(["one", "one", "steps"])
    token_major = rng.random() < 0.25
    if sort == "f32":     # any width, odd ones too
        c = _layer("", "f32", _log(rng, 16, 4096), _log(rng, 48, 1024), rng.choice([5, 8, 16, 32, 128]),
                   rng.choice([1, 2, 3, 4]), _log(rng, 30, 1024), rng.random() < 0.7, zipf, 0.05, calls,
                   dbias=rng.random() < 0.3, token_major=token_major)
        if rng.random() < 0.7:
            c["d"], c["F"] = (c["d"] + 3) // 4 * 4, (c["F"] + 3) // 4 * 4
        _fit(c, 18.0 * 2048 * 4 * 512 * 1024)
    elif sort == "ragged":   # widths that are multiples of 8 but not of 256
        width = lambda: 8 * _log(rng, 5, 256)  # noqa: E731
        c = _layer("", "bf16", _log(rng, 16, 8192), width(), rng.choice([6, 16, 60, 64, 128]), rng.choice([2, 4, 6]),
                   width(), rng.random() < 0.7, zipf, sigma, calls, dbias=rng.random() < 0.3, token_major=token_major)
        c["d"] += 8 if c["d"] % 256 == 0 else 0
        _fit(c, 18.0 * 3001 * 6 * 1000 * 704)
    else:
        d, F, E = rng.choice([512, 768, 1024, 2048, 2048]), rng.choice([256, 512, 768, 768, 1280]), rng.choice([64, 128, 128, 256, 384])
        while E * d * F > 128 * 2048 * 768:
            E //= 2
        c = _layer("", "bf16", _log(rng, 1, 131072) if sort == "forward" else _log(rng, 48, 65536), d, E,
                   rng.choice([2, 4, 8, 8]), F, sort == "train", zipf, sigma, calls, agree=sort == "forward" and rng.random() < 0.5,
                   dbias=sort == "train" and rng.random() < 0.3, token_major=token_major)
        _fit(c, 18.0 * 65536 * 8 * 2048 * 768)
        c["T"] = min(c["T"], 131072 * 8 // c["K"], 131072 * 2048 // d)
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------------------- layer
class _State:
    pass


def _prepare_layer(c, seed):
    s = _State()
    sh = synth.LayerShape(T=c["T"], d=c["d"], E=c["E"], K=c["K"], F=c["F"], act=c["act"], sigma=c["sigma"],
                          zipf_s=c["zipf"] or None, seed=seed)
    L = 3 if c["token_major"] else 1          # a token-major record of three layers; this layer is the middle one
    s.D = r3.desc(sh.T, sh.d, sh.E, sh.K, sh.F, sh.act, idx_token_stride=L * sh.K if c["token_major"] else 0)
    a = r3.act_dtype(s.D)
    s.x, s.Wr, s.Wg, s.Wu, s.Wd = (synth.draw(sh, k, "cuda").to(a) for k in ("x", "Wr", "Wg", "Wu", "Wd"))
    s.dy = synth.draw(sh, "dy", "cuda").to(a) if c["backward"] else None
    s.bias = synth.draw(sh, "bias", "cuda")
    # what the rollout's router saw: the training logits plus the inference engine's noise
    Wr64 = s.Wr.double()
    lg = torch.cat([s.x[i:i + 16384].double() @ Wr64 for i in range(0, sh.T, 16384)])
    if s.bias is not None:
        lg += s.bias.double()
    s.s_infer = (lg + synth.draw(sh, "noise", "cuda").double()).float()
    rec = torch.zeros(sh.T, L, sh.K, dtype=torch.uint8 if sh.E <= 256 else torch.int16, device="cuda")
    if sh.E > 256:
        rec = rec.view(torch.uint16)
    s.record = rec[:, L // 2]
    s.buf = r3.LayerBuffers(s.D, backward=c["backward"], gathered_copy=False)
    s.agree = torch.zeros(2, dtype=torch.int64, device="cuda") if c["agree"] else None
    s.dbias = torch.zeros(sh.E, dtype=torch.float32, device="cuda") if c["dbias"] and c["backward"] else None
    s.forward = r3.forward if c["calls"] == "steps" else r3.forward_one_call
    s.backward = c["backward"]
    s.wide = sh.E > 256
    return s


def _run_layer(s):
    b = s.buf
    r3.record_topk(s.D, s.s_infer, s.record, b.status)
    if s.agree is not None:
        s.agree.zero_()
    s.forward(b, s.x, s.Wr, s.record, s.Wg, s.Wu, s.Wd, bias=s.bias, agree_out=s.agree)
    # uint16 ids are handed on as int16: the same bits, in a type every consumer takes
    rec = s.record.view(torch.int16) if s.wide else s.record
    out = {"record": rec, "y": b.y, "gates": b.gates, "counts": b.counts, "offsets": b.offsets, "perm": b.perm,
           "inv_perm": b.inv_perm, "status": b.status}
    if s.agree is not None:
        out["agreement"] = s.agree.double() / s.D.T      # share of tokens, mean shared experts
    if s.backward:
        r3.backward(b, s.dy, s.x, s.Wr, s.record, s.Wg, s.Wu, s.Wd, dbias=s.dbias)
        out.update(dx=b.dx, dW_r=b.dW_r, dW_gate=b.dW_gate, dW_up=b.dW_up, dW_down=b.dW_down)
        if s.dbias is not None:
            out["dbias"] = s.dbias
    return out


def _work_layer(c):
    T, d, E, K, F = c["T"], c["d"], c["E"], c["K"], c["F"]
    eb = 2 if c["act"] == "bf16" else 4
    ib = 1 if E <= 256 else 2
    hit = E * (1.0 - (1.0 - K / E) ** T)      # experts some token chose (under a balanced load)
    b = T * E * 4 + T * K * ib                # the record from the rollout's logits
    b += 2 * T * d * eb + d * E * eb + T * K * 4 + 3 * hit * d * F * eb
    b += 2 * T * K * 4 + (2 * E + 1) * 4      # inverse permutation, permutation, counts, offsets
    f = 2.0 * T * d * E + 6.0 * T * K * d * F
    if c["backward"]:
        b += 2 * T * d * eb + d * E * 4 + 3 * E * d * F * 4      # dy, dx and the weight gradients
        f += 2.0 * T * d * E + 2.0 * T * d * K + 12.0 * T * K * d * F
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------------------------------------- cache
def _prepare_cache(c, seed):
    s = _State()
    L, T, K, E, P = c["L"], c["T"], c["K"], c["E"], c["P"]
    lens, shared, table, used = synth.rollout_batch(T, P, group=c["group"], seed=seed % (1 << 31))
    num_pages = T // P * 5 // 4 + 128         # the engine's page pool; a batch fills most of it
    assert used <= num_pages
    start = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    seq = np.concatenate([np.full(int(n - h), i, np.int32) for i, (n, h) in enumerate(zip(lens, shared))])
    pos = np.concatenate([np.arange(h, n, dtype=np.int32) for n, h in zip(lens, shared)])
    s.n = len(seq)
    g = torch.Generator(device="cuda").manual_seed(seed)
    s.dt = torch.uint8 if E <= 256 else torch.int16
    ids = torch.randint(0, E, (L, s.n, K), generator=g, device="cuda", dtype=torch.int16).to(s.dt)
    as_ids = (lambda t: t) if E <= 256 else (lambda t: t.view(torch.uint16))
    s.new = as_ids(ids)
    s.pages = as_ids(torch.zeros((num_pages, P, L, K), dtype=s.dt, device="cuda"))
    s.out = as_ids(torch.zeros((L, T, K), dtype=s.dt, device="cuda"))
    s.table, s.seq, s.pos, s.start = (torch.from_numpy(a).to("cuda") for a in (table, seq, pos, start))
    s.status = torch.zeros(1, dtype=torch.int32, device="cuda")
    s.K = K
    return s


def _run_cache(s):
    r3.mask_cache_append(s.pages, s.table, s.seq, s.pos, s.new, s.n * s.K, s.K, s.status)
    r3.mask_cache_gather(s.pages, s.table, s.start, s.out, s.status)
    return {"pages": s.pages.view(s.dt), "out": s.out.view(s.dt), "status": s.status}


def _work_cache(c):
    b = 1 if c["E"] <= 256 else 2
    # about three quarters of the tokens have pages of their own (the rest share a prompt's)
    return {"bytes": (2 + 1.5) * c["L"] * c["T"] * c["K"] * b + 8 * c["T"], "flops": 0}


# ----------------------------------------------------------------------------------------------------- diagnostics
def _prepare_diag(c, seed):
    s = _State()
    L, T, K, E, n = c["L"], c["T"], c["K"], c["E"], c["n"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.uint8 if E <= 256 else torch.int16
    shape = (T, L) if c["token_major"] else (L, T)

    def sets(*lead):   # K distinct ids per router: one of each of K strata
        w = E // K
        r = torch.randint(0, w, (*lead, K), generator=g, device="cuda", dtype=torch.int16)
        return r + w * torch.arange(K, device="cuda", dtype=torch.int16)
    a = sets(*shape)
    # about one router in ten differs, mostly in one choice
    hit = torch.rand(*shape, K, generator=g, device="cuda") < 0.0125
    b = torch.where(hit, sets(*shape), a)
    as_ids = (lambda t: t.to(dt).contiguous()) if E <= 256 else (lambda t: t.contiguous().view(torch.uint16))
    s.a, s.b = as_ids(a), as_ids(b)
    s.D = r3.desc(T, 16, E, K, 16, idx_token_stride=L * K if c["token_major"] else 0)
    s.L, s.layer_stride = L, K if c["token_major"] else T * K
    s.hist = torch.zeros(K + 1, dtype=torch.int64, device="cuda")
    s.tc, s.tr = (torch.empty(T, dtype=torch.int32, device="cuda") for _ in range(2))
    cuts = sorted(set(list(range(0, T, 2048)) + [T]))
    s.so = torch.tensor(cuts, dtype=torch.int32, device="cuda")
    s.sm = torch.empty(len(cuts) - 1, dtype=torch.float64, device="cuda")
    s.li = torch.log(torch.rand(n, generator=g, device="cuda").clamp_min(1e-4))
    s.lt = s.li + 0.05 * torch.randn(n, generator=g, device="cuda")
    s.kl = torch.zeros(1, dtype=torch.float64, device="cuda")
    s.frac = torch.zeros(len(TAUS), dtype=torch.float64, device="cuda")
    s.ws = torch.empty(256 << 10, dtype=torch.uint8, device="cuda")
    return s


def _run_diag(s):
    s.hist.zero_()
    r3.routing_diff(s.D, s.L, s.a, s.b, s.layer_stride, s.hist, s.tc, s.tr, s.so, s.sm)
    r3.policy_discrepancy(s.lt, s.li, TAUS, s.kl, s.frac, s.ws)
    return {"hist": s.hist, "token_choices": s.tc, "token_routers": s.tr, "seq_mean": s.sm, "kl": s.kl, "frac": s.frac}


def _work_diag(c):
    b = 1 if c["E"] <= 256 else 2
    return {"bytes": 2 * c["L"] * c["T"] * c["K"] * b + 8 * c["T"] + 8 * c["n"], "flops": 0}


# -------------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    return case["kind"], {"layer": _prepare_layer, "cache": _prepare_cache, "diag": _prepare_diag}[case["kind"]](case, seed)


def run(state):
    kind, s = state
    return {"layer": _run_layer, "cache": _run_cache, "diag": _run_diag}[kind](s)


def work(case):
    return {"layer": _work_layer, "cache": _work_cache, "diag": _work_diag}[case["kind"]](case)


def tolerance(case):
    if case["kind"] == "cache":
        return "exact"
    if case["kind"] == "diag":
        # counts are exact; kl is a float64 sum of up to ten million terms
        return {"rel": 1e-11, "max": 1e-10}
    # against the same layer in float64 (every output, all training cases): float32 up to rel 1.1e-6, max 1e-5; bf16 up
    # to rel 3.5e-3 (dx), max 0.14 (one element of a weight gradient of an expert with a handful of rows)
    if case["act"] == "f32":
        return {"rel": 5e-6, "max": 5e-5}
    return {"rel": 1.2e-2, "max": 0.5}
