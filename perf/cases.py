"""The work that users of libpsattn have it do, as measurable cases.

A case is a plain dict: what is called (`kind`), the element type, the heads, and a recipe for the sample
table (length ranges, packing, seed of the lengths).  `prepare` makes what a training program has in hand
before the call, `run` is one pass through the public entry points, `work` the bytes and operations such a
pass cannot do without, `tolerance` how far another correct implementation may be off.

Kinds
  step     one training step of an attention layer: block mask, forward, backward, release of the mask
  rope     the same on a kept block mask with the rotary embedding inside the op, any number of responses
  forward  forward only (the frozen reference policy of DPO needs no backward), kept block mask
  logprob  response log-probabilities, DPO loss, gradient of the logits
  layer    a whole attention layer, forward and backward, kept block mask
"""
import math

import numpy as np
import torch

import paper_2410_20305_amd as ps
from paper_2410_20305_amd.layer import Layer

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


# ------------------------------------------------------------------ sample tables
def _table(case):
    """offset, prompt length, response lengths per sample and the buffer's length in tokens.  `rows` > 0: samples
    are packed in order into that many rows of `row_len` tokens, the rest of a row is padding."""
    rng = np.random.default_rng(case["table"])
    draw = lambda lo, hi: int(rng.integers(lo, hi, endpoint=True))
    off, prompt, resp = [], [], []
    at, row = 0, 0
    rows, row_len = case.get("rows", 0), case.get("row_len", 0)
    while rows or len(off) < case["n"]:
        p = draw(case["p_lo"], case["p_hi"])
        r = [draw(case["c_lo"], case["c_hi"]) for _ in range(case.get("k", 2))]
        size = p + sum(r)
        if rows and at + size > (row + 1) * row_len:
            row += 1
            at = row * row_len
            if row == rows:
                break
        off.append(at)
        prompt.append(p)
        resp.append(r)
        at += size
    return off, prompt, resp, rows * row_len if rows else at


def _pairs(prompt, resp):
    """(query, key) pairs that the mask allows."""
    tri = lambda n: n * (n + 1) // 2
    return sum(tri(p) + sum(r * p + tri(r) for r in rs) for p, rs in zip(prompt, resp))


def _logit_rows(prompt, resp):
    """Logits rows that predict a response token: the last prompt row and every response row but its last."""
    return sum((1 if p else 0) + sum(r - 1 for r in rs) for p, rs in zip(prompt, resp))


# ------------------------------------------------------------------ the cases
def _case(name, kind, dtype, hq, hkv, d, table, p, c, n=0, rows=0, row_len=0, k=2, **more):
    case = dict(name=name, kind=kind, dtype=dtype, hq=hq, hkv=hkv, d=d, table=table, n=n, rows=rows, row_len=row_len,
                k=k, p_lo=p[0], p_hi=p[1], c_lo=c[0], c_hi=c[1])
    case.update(more)
    return {key: v for key, v in case.items() if v is not None}


def listed():
    return [
        # the smallest call: one fp32 sample on one head, as in a numerics check; latency and launches are all there is
        _case("tiny_fp32_step", "step", "f32", 1, 1, 64, 0, (96, 96), (24, 40), n=1),
        # one short dialogue (about 190 tokens) per device: launches, host work and a nearly empty chip
        _case("short_sample_step", "step", "bf16", 32, 8, 128, 7, (90, 130), (20, 60), n=1),
        # a batch of moderate single-turn samples, unpacked
        _case("moderate_batch_step", "step", "bf16", 32, 8, 128, 2, (256, 1024), (64, 384), n=8),
        # summarisation-like: long prompts, short answers
        _case("long_prefix_step", "step", "bf16", 32, 8, 128, 3, (1024, 3072), (32, 192), n=16),
        # many short samples packed into rows: block-diagonal mask, most tiles partial
        _case("packed_short_step", "step", "bf16", 32, 8, 128, 4, (32, 256), (32, 256), rows=8, row_len=8192),
        # long multi-turn context packed into rows: the largest attention step
        _case("packed_long_step", "step", "bf16", 64, 8, 128, 5, (2048, 6144), (128, 1024), rows=4, row_len=16384),
        # four responses per prompt (several candidates against one prompt), rotary embedding inside the op
        _case("four_responses_rope", "rope", "bf16", 32, 8, 128, 11, (200, 1500), (50, 400), n=12, k=4),
        # the frozen reference policy: forward only, packed rows of moderate samples
        _case("reference_forward", "forward", "bf16", 32, 8, 128, 12, (256, 1024), (64, 384), rows=4, row_len=4096),
        # the other head size: a small model's heads of 64
        _case("head64_step", "step", "bf16", 32, 8, 64, 13, (128, 512), (32, 192), n=8),
        # loss head of the long packed batch, vocabulary 32 000
        _case("logprob_head", "logprob", "bf16", None, None, None, 5, (2048, 6144), (128, 1024), rows=4, row_len=16384,
              vocab=32000),
        # loss head in fp32 with an odd vocabulary (rows that are not 16-byte aligned)
        _case("logprob_odd_vocab_fp32", "logprob", "f32", None, None, None, 2, (256, 1024), (64, 384), n=8, vocab=50257),
        # a whole attention layer on four samples of prompt 1024 and two answers of 128
        _case("attention_layer", "layer", "bf16", 32, 8, 128, 1, (1024, 1024), (128, 128), n=4, hidden=4096),
    ]


# a drawn case costs no more than the largest listed one
_MOST_FLOPS = 14 * 128 * 64 * 134_816_577
_MOST_LOGITS = 65_536 * 32_000


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    while True:
        kind = rng.choice(("step", "step", "step", "rope", "forward", "logprob", "layer", "head64", "fp32"))
        table = rng.randrange(1 << 30)
        p_hi, c_hi = _log(rng, 64, 6144), _log(rng, 32, 1024)
        p, c = (max(1, p_hi // rng.choice((2, 3, 8))), p_hi), (max(1, c_hi // rng.choice((2, 4, 8))), c_hi)
        hq, hkv = rng.choice(((32, 8), (32, 8), (64, 8), (16, 16), (24, 6), (28, 4)))
        k = rng.choice((1, 2, 2, 2, 4, 6)) if kind in ("step", "rope", "forward") else 2
        rows = rng.choice((0, 0, rng.randint(1, 8)))
        if rows:
            row_len = max(_log(rng, 1024, 16384), p_hi + k * c_hi)
            lay = dict(rows=rows, row_len=row_len)
        else:
            lay = dict(n=_log(rng, 1, 48))
        if kind == "fp32":
            hq, hkv = rng.choice(((1, 1), (2, 1), (4, 2), (8, 2)))
            case = _case(None, "step", "f32", hq, hkv, rng.choice((64, 128)), table, (rng.randint(5, 60), _log(rng, 64, 300)),
                         (rng.randint(1, 20), _log(rng, 24, 150)), n=rng.randint(1, 3))
        elif kind == "head64":
            case = _case(None, "step", "bf16", hq, hkv, 64, table, (rng.randint(20, 60), _log(rng, 64, 700)),
                         (rng.randint(5, 30), _log(rng, 32, 250)), n=rng.randint(1, 10))
        elif kind == "logprob":
            vocab = rng.choice((32000, 32000, _log(rng, 1000, 130000), _log(rng, 1000, 130000)))
            case = _case(None, "logprob", rng.choice(("bf16", "bf16", "f32")), None, None, None, table, p, c, vocab=vocab, **lay)
        elif kind == "layer":
            case = _case(None, "layer", "bf16", 32, 8, 128, table, p, c, hidden=rng.choice((2048, 4096)), **lay)
        else:
            case = _case(None, kind, "bf16", hq, hkv, 128, table, p, c, k=k, **lay)
        _, prompt, resp, T = _table(case)
        if not prompt or T < 64:
            continue
        if kind == "logprob":
            if T * case["vocab"] * (2 if case["dtype"] == "f32" else 1) <= _MOST_LOGITS:
                return case
        elif kind == "layer":
            if T <= 20_000 and work(case)["flops"] <= _MOST_FLOPS // 2:
                return case
        elif T <= 65_536 and work(case)["flops"] <= _MOST_FLOPS:
            return case


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    _, prompt, resp, T = _table(case)
    if case["kind"] == "logprob":
        e, v = (2 if case["dtype"] == "bf16" else 4), case["vocab"]
        rows = _logit_rows(prompt, resp)
        # the logits rows that predict something are read once, the whole gradient is written once
        return {"bytes": (rows + T) * v * e + 8 * T, "flops": 5 * rows * v}
    e, hq, hkv, d = (2 if case["dtype"] == "bf16" else 4), case["hq"], case["hkv"], case["d"]
    q, kv, stats = T * hq * d * e, T * hkv * d * e, 4 * T * hq
    n = _pairs(prompt, resp) * hq * d
    if case["kind"] == "forward":
        return {"bytes": 2 * q + 2 * kv + stats, "flops": 4 * n}
    if case["kind"] == "layer":
        h = case["hidden"]
        weights = h * d * (2 * hq + 2 * hkv)
        # X, dY, Y, dX once, weights and their gradients once; three products per weight
        return {"bytes": 4 * T * h * e + 2 * weights * e, "flops": 14 * n + 6 * T * weights}
    rotated = q + kv if case["kind"] == "rope" else 0
    # Q, K, V, dO read, O, LSE, dQ, dK, dV written (and the rotated Q, K, which are results too)
    return {"bytes": 4 * q + 4 * kv + stats + rotated, "flops": 14 * n}


def tolerance(case):
    # each about four times what the path shows against the same sums in 64 bits
    if case["kind"] == "logprob":
        # fp32: one exponential per element, 1.1e-7; bf16: one rounding of the gradient, 1.0e-3
        return {"rel": 1e-6} if case["dtype"] == "f32" else {"rel": 4e-3}
    if case["dtype"] == "f32":
        # sums of fp32 products: 4e-7 (head size 64, 168 tokens) to 8e-7 (head size 128, 1200 tokens)
        return {"rel": 4e-6}
    # probabilities and score gradients enter the second products as bf16: 1.6e-3 to 2.5e-3
    return {"rel": 1e-2}


# ------------------------------------------------------------------ preparing and running
def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    off, prompt, resp, T = _table(case)
    dt = _DTYPES[case["dtype"]]
    randn = lambda *shape, scale=1.0: torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(scale).to(dt)
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in resp])]).astype(np.int32)
    flat = np.array([x for r in resp for x in r], dtype=np.int32)
    s = dict(kind=case["kind"], T=T, off=np.array(off, dtype=np.int32), prompt=np.array(prompt, dtype=np.int32), ptr=ptr, resp=flat)
    if case["kind"] == "logprob":
        vocab = case["vocab"]
        s["plan"] = ps.LogprobPlan(off, prompt, ptr, flat, T)
        logits = torch.empty((T, vocab), dtype=dt, device="cuda")
        for t in range(0, T, 8192):  # in pieces: the draw is made in fp32
            logits[t:t + 8192] = randn(min(8192, T - t), vocab, scale=3.0)
        s["logits"] = logits
        s["ids"] = torch.randint(0, vocab, (T,), generator=gen, device="cuda", dtype=torch.int32)
        n = len(flat)
        s["ref_logp"] = -10.0 * torch.rand(n, generator=gen, device="cuda") - 10.0
        s["row_lse"] = torch.zeros(T, device="cuda")
        s["logp"] = torch.empty(n, device="cuda")
        s["dlogits"] = torch.empty_like(logits)
        return s
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    s["scale"] = 1.0 / math.sqrt(d)
    build = lambda: ps.psattn_build_meta_multi(s["off"], s["prompt"], ptr, flat, T)
    if case["kind"] == "layer":
        h = case["hidden"]
        s["meta"] = build()
        s["rope"] = ps.Rope(d, 10000.0, s["meta"].positions()[1])
        s["layer"] = Layer(h, hq, hkv, d)
        s["weights"] = (randn(hq * d, h, scale=h ** -0.5), randn(hkv * d, h, scale=h ** -0.5), randn(hkv * d, h, scale=h ** -0.5),
                        randn(h, hq * d, scale=(hq * d) ** -0.5))
        s["X"], s["dY"] = randn(T, h), randn(T, h)
        s["ws"] = torch.empty(s["layer"].workspace_bytes(s["meta"]), dtype=torch.uint8, device="cuda")
        s["Y"] = torch.empty_like(s["X"])
        s["grads"] = tuple(torch.empty_like(t) for t in (s["X"],) + s["weights"])
        return s
    s["two"] = case.get("k", 2) == 2
    s["chosen"], s["rejected"] = (flat[0::2].copy(), flat[1::2].copy()) if s["two"] else (None, None)
    s["Q"], s["K"], s["V"], s["dO"] = randn(T, hq, d), randn(T, hkv, d), randn(T, hkv, d), randn(T, hq, d)
    s["O"], s["LSE"] = torch.empty_like(s["Q"]), torch.empty((hq, T), device="cuda")
    if case["kind"] == "forward":
        s["meta"] = build()
        return s
    s["dQ"], s["dK"], s["dV"] = torch.empty_like(s["Q"]), torch.empty_like(s["K"]), torch.empty_like(s["V"])
    meta = build()
    s["ws"] = torch.empty(ps.psattn_bwd_workspace_bytes(meta, hq, hkv, d), dtype=torch.uint8, device="cuda")
    if case["kind"] == "rope":
        s["meta"] = meta
        s["rope"] = ps.Rope(d, 500000.0, meta.positions()[1])
        s["Qr"], s["Kr"] = torch.empty_like(s["Q"]), torch.empty_like(s["K"])
    else:
        meta.free_async()  # a step builds its own
    return s


def run(s):
    kind = s["kind"]
    if kind == "logprob":
        ps.psattn_logprob_fwd(s["plan"], s["logits"], s["ids"], row_lse=s["row_lse"], resp_logp=s["logp"])
        loss, d_logp = ps.psattn_dpo_loss(s["logp"], s["ref_logp"], 0.1)
        ps.psattn_logprob_bwd(s["plan"], s["logits"], s["ids"], s["row_lse"], d_logp, dlogits=s["dlogits"])
        return s["row_lse"], s["logp"], loss, d_logp, s["dlogits"]
    if kind == "layer":
        args = (s["meta"], s["rope"], s["scale"], s["X"]) + s["weights"]
        s["layer"].forward(*args, s["ws"], Y=s["Y"])
        s["layer"].backward(*args, s["dY"], s["ws"], grads=s["grads"])
        return (s["Y"],) + s["grads"]
    Q, K, V, O, LSE, scale = s["Q"], s["K"], s["V"], s["O"], s["LSE"], s["scale"]
    if kind == "forward":
        ps.psattn_fwd(s["meta"], Q, K, V, scale, O=O, LSE=LSE)
        return O, LSE
    grads = dict(dQ=s["dQ"], dK=s["dK"], dV=s["dV"], workspace=s["ws"])
    if kind == "rope":
        ps.psattn_fwd_rope(s["meta"], s["rope"], Q, K, V, scale, O=O, LSE=LSE, Qr=s["Qr"], Kr=s["Kr"])
        ps.psattn_bwd_rope(s["meta"], s["rope"], s["Qr"], s["Kr"], V, O, s["dO"], LSE, scale, **grads)
        return O, LSE, s["Qr"], s["Kr"], s["dQ"], s["dK"], s["dV"]
    if s["two"]:
        meta = ps.psattn_build_meta(s["off"], s["prompt"], s["chosen"], s["rejected"], s["T"])
    else:
        meta = ps.psattn_build_meta_multi(s["off"], s["prompt"], s["ptr"], s["resp"], s["T"])
    ps.psattn_fwd(meta, Q, K, V, scale, O=O, LSE=LSE)
    ps.psattn_bwd(meta, Q, K, V, O, s["dO"], LSE, scale, **grads)
    meta.free_async()
    return O, LSE, s["dQ"], s["dK"], s["dV"]
