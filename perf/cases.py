"""The work that programs have this decoder do, as cases to measure.

Two kinds of case:

- "expand": one decoder step (recurrence, vocabulary projection, row merge)
  on explicit rows through Decoder.debug_expand: new states, log-sum-exp,
  best k log-probabilities and tokens of every row. This is the step a
  program takes to score or extend given prefixes.
- "decode": a whole streaming beam search through Decoder.reset, submit, run
  and collect_arrays, laid out densely by input and rank as a reranker or a
  writer of n-best lists takes it.

Shapes are those of synthgen.configs: a tiny search (|V| = 1000, d = 64), a
parsing-like one (|V| = 256, d = 256), and machine translation (|V| = 32000
or 64000, d = 1024, fp32 and bf16, also with a KV state and attention).
Weights are N(0, 1/d), lengths uniform or lognormal(3.2, 0.5), as there.
"""
import math

import numpy as np
import torch

from paper_2010_02164_amd import Decoder

TINY = dict(V=1000, d=64, dtype="f32", k=4, M=4, delta=1.5, beta=0.5, lengths="uniform", lo=4, hi=20, max_len=32)
PARSE = dict(V=256, d=256, dtype="f32", k=5, M=3, delta=2.0, beta=0.5, lengths="uniform", lo=5, hi=60, max_len=128)
MT = dict(V=32000, d=1024, dtype="f32", k=5, M=5, delta=1.5, beta=1.0, lengths="lognormal", lo=3, hi=200, max_len=0)
WIDE = dict(MT, dtype="bf16", k=10, M=4)
KV = dict(MT, dtype="bf16", V=64000, M=4)


def _expand(name, shape, rows):
    return dict(name=name, kind="expand", rows=rows, V=shape["V"], d=shape["d"], dtype=shape["dtype"], k=shape["k"])


def _decode(name, shape, sched, N, n, kv=0, attn=False):
    return dict(shape, name=name, kind="decode", sched=sched, N=N, n=n, eps=0.25, kv=kv, attn=attn)


def listed():
    return [
        # The smallest call: a handful of prefixes on the tiny model, where
        # launches and copies count.
        _expand("step_tiny_f32", TINY, 7),
        # A parsing batch: many rows, a small vocabulary.
        _expand("step_parse_f32", PARSE, 2126),
        # Translation in fp32: the stragglers at the end of a batch, an
        # ordinary step (ragged), and a full batch of 128 beams of 5.
        _expand("step_mt_f32_tail", MT, 21),
        _expand("step_mt_f32", MT, 193),
        _expand("step_mt_f32_full", MT, 640),
        # Translation in bf16: an ordinary step over the large vocabulary,
        # and a full batch of 512 beams of 10.
        _expand("step_mt_bf16", KV, 389),
        _expand("step_mt_bf16_full", WIDE, 5120),
        # Whole searches: a short tiny one (an interactive request), ...
        _decode("decode_tiny_f32", TINY, "var_stream", 64, 8),
        # ... a corpus of parses with the pool of cached beams, ...
        _decode("decode_parse_f32", PARSE, "var_cap", 2048, 1024),
        # ... the headline translation workload's batch in fp32, ...
        _decode("decode_mt_f32", MT, "var_stream", 256, 128),
        # ... wide bf16 beams with every live beam expanded at each step, ...
        _decode("decode_mt_bf16", WIDE, "var_fifo", 256, 128),
        # ... and the length-dependent step: KV state and self-attention.
        _decode("decode_attn_bf16", KV, "var_stream", 48, 32, kv=6, attn=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: rows 1 to 5120, |V| 200 to 64000,
    d 64 to 1024, k 1 to 12, both types, every kind of search listed; a
    drawn step stays below the largest listed one's work, a drawn search
    below the listed translation searches'."""
    dtype = rng.choice(["f32", "bf16"])
    d = rng.choice([64, 192, 256, 512, 1024]) if dtype == "f32" else rng.choice([128, 256, 384, 512, 1024])
    k = rng.choice([1, 3, 4, 5, 8, 10, 12])
    if rng.random() < 0.6:
        V = _log_int(rng, 200, 64000)
        most = 640 * 32000 * 1024 if dtype == "f32" else 5120 * 32000 * 1024
        rows = _log_int(rng, 1, min(5120, max(2, most // (V * d))))
        return dict(kind="expand", rows=rows, V=V, d=d, dtype=dtype, k=k)
    n = _log_int(rng, 4, 128)
    kv = rng.choice([0, 0, 2, 6]) if dtype == "bf16" else 0
    attn = kv > 0 and d != 384 and d != 128 and rng.random() < 0.5
    short = rng.random() < 0.5
    return dict(kind="decode", V=_log_int(rng, 200, 16000), d=d, dtype=dtype, k=k, M=rng.choice([k, max(1, k - 2)]),
                delta=rng.choice([1.5, 2.0]), beta=rng.choice([0.5, 1.0]),
                lengths="uniform" if short else "lognormal", lo=4 if short else 3, hi=20 if short else 100,
                max_len=32 if short else 0, sched=rng.choice(["var_stream", "var_fifo", "var_cap", "fixed_stream"]),
                N=_log_int(rng, n, min(160, 4 * n)), n=n, eps=rng.choice([0.125, 0.25, 0.5]), kv=kv, attn=attn)


def _weights(case, g):
    V, d = case["V"], case["d"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    s = d ** -0.5

    def w(*shape):
        return (torch.randn(*shape, generator=g, device="cuda") * s).to(dt)

    kv = w(case["kv"], 2, d, d) if case.get("kv") else None
    return w(d, d), w(V, d), w(V, d), kv


def _lengths(case, seed):
    r = np.random.default_rng(seed)
    if case["lengths"] == "uniform":
        L = r.integers(case["lo"], case["hi"] + 1, case["N"])
    else:
        L = np.clip(np.rint(r.lognormal(3.2, 0.5, case["N"])), case["lo"], case["hi"]).astype(np.int64)
    ml = np.full(case["N"], case["max_len"]) if case["max_len"] else (12 * L + 100) // 10
    return L.astype(np.int32), ml.astype(np.int32)


def _cap(case):
    return case["max_len"] or (12 * case["hi"] + 100) // 10


def _inputs(case, seed):
    """Weights and inputs of a case, made from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    W = _weights(case, g)
    dt, d = W[0].dtype, case["d"]
    if case["kind"] == "expand":
        R = case["rows"]
        h = torch.tanh(0.5 * torch.randn(R, d, generator=g, device="cuda")).to(dt)
        r = np.random.default_rng(seed)
        return W, (h, r.integers(0, case["V"], R).astype(np.int32), r.integers(1, 40, R).astype(np.int32),
                   r.integers(3, 40, R).astype(np.int32))
    h0 = torch.randn(case["N"], d, generator=g, device="cuda").to(dt)
    return W, (h0,) + _lengths(case, seed)


def prepare(case, seed):
    (W_h, E, W_out, W_kv), x = _inputs(case, seed)
    k = case["k"]
    if case["kind"] == "expand":
        dec = Decoder(W_h, E, W_out, beta=1.0, k=k, n=-(-case["rows"] // k), max_len_cap=8, max_inputs=1)
        return dict(case=case, dec=dec, x=x)
    dec = Decoder(W_h, E, W_out, W_kv=W_kv, beta=case["beta"], k=k, n=case["n"], eps=case["eps"], delta=case["delta"],
                  M=case["M"], sched=case["sched"], max_len_cap=_cap(case), max_inputs=case["N"], attn=case["attn"],
                  pool=2 * case["n"] if case["sched"] == "var_cap" else None)
    return dict(case=case, dec=dec, x=x, tokens=np.zeros(case["N"] * k * _cap(case), np.int32))


def run(state):
    case, dec = state["case"], state["dec"]
    if case["kind"] == "expand":
        h, lse, lp, tok = dec.debug_expand(*state["x"])
        return dict(h=h, lse=lse, lp=lp, tok=tok)
    dec.reset()
    dec.submit(*state["x"])
    dec.run()
    return _dense(dec.collect_arrays(), case["N"], case["k"], _cap(case), state["tokens"])


def _dense(a, N, k, cap, tokens):
    """The n-best lists as dense arrays: scores [N, k] (a list shorter than k
    repeats its last score, as a reranker of fixed width takes it), lengths
    and statuses [N, k] (0 past the list's end) and
    tokens [N, k, cap]."""
    slot = a["input"] * k + a["rank"]
    count = np.bincount(a["input"], minlength=N)
    score = np.zeros(N * k)
    length = np.zeros(N * k, np.int32)
    status = np.zeros(N * k, np.int32)
    score[slot], length[slot], status[slot] = a["score"], a["length"], a["status"]
    last = np.minimum(np.arange(k)[None, :], count[:, None] - 1)
    score = np.take_along_axis(score.reshape(N, k), last, 1)
    tokens.fill(0)
    n_tok = len(a["tokens"])
    tokens[np.repeat(slot * cap - a["tok_offset"], a["length"]) + np.arange(n_tok)] = a["tokens"]
    return dict(score=score, length=length.reshape(N, k), status=status.reshape(N, k),
                tokens=tokens.reshape(N, k, cap))


def _mean_len(case):
    return (case["lo"] + case["hi"]) / 2 if case["lengths"] == "uniform" else math.exp(3.2 + 0.125)


def work(case):
    """Weights and inputs read once, outputs written once, and the products
    of every expansion. A search expands about k candidates a step for as
    many steps as its length; its weights are read once for each step of the
    longest output (a step needs the one before)."""
    V, d, k = case["V"], case["d"], case["k"]
    es = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "expand":
        R = case["rows"]
        return dict(bytes=(V * d + d * d) * es + R * d * es * 3 + R * (8 + 12 * k), flops=2.0 * R * d * (V + d))
    mean = _mean_len(case)
    rows = case["N"] * k * mean
    longest = case["hi"] if case["lengths"] == "uniform" else min(case["hi"], math.exp(3.2 + 0.5 * 2.5))
    planes = 2 * case["kv"]
    b = longest * (V * d + d * d * (1 + planes)) * es + rows * d * es * 4 + rows * planes * d * 2
    f = 2.0 * rows * d * (V + d + planes * d)
    if case["attn"]:
        b += rows * planes * d * mean / 2 * 2
        f += 2.0 * rows * planes * d * mean / 2
    return dict(bytes=b, flops=f)


def tolerance(case):
    """Steps: fp32 sums over d products and a log-sum-exp over |V| terms;
    equal in another order to about 2e-7 of their norm, so that of two
    tokens whose logits differ by less either may come first. bf16 states
    are rounded once: a state whose exact value lies at a rounding boundary
    may differ by one bf16 step. Searches: such a pair of candidates within
    rounding of each other (or of the pruning threshold) may be decided
    either way, after which that input's lower ranks differ."""
    if case["kind"] == "expand":
        if case["dtype"] == "f32":
            return {"rel": 2e-6, "max": 4e-5, "differ": 5e-3}
        return {"rel": 1e-4, "max": 8e-3, "differ": 5e-3}
    return {"rel": 5e-3, "max": 0.1, "differ": 0.01}


# ---------------------------------------------------------------- 64 bits
def _bf16(x):
    """64-bit values rounded once to bf16's 8 significant bits (a conversion
    through 32 bits rounds twice)."""
    m, e = torch.frexp(x)
    return torch.ldexp(torch.round(m * 256), e - 8)


def _step64(case, W, h, y, bias, x_of=None):
    """New states (and, for bf16, their stored values), log-sum-exp and
    logits of one decoder step in 64 bits."""
    W_h, E, W_out = (w.double() for w in W[:3])
    exact_h = torch.tanh(h.double() @ W_h.T + E[y])
    hs = _bf16(exact_h) if case["dtype"] == "bf16" else exact_h
    z = (hs if x_of is None else x_of(hs)) @ W_out.T
    z[:, 0] += bias
    return exact_h, hs, torch.logsumexp(z, 1), z


def exact(case, seed):
    if case["kind"] == "expand":
        W, (h, y, t, Lx) = _inputs(case, seed)
        bias = torch.from_numpy((t - Lx).astype(np.float64)).cuda()
        eh, _, lse, z = _step64(case, W, h, torch.from_numpy(y).cuda().long(), bias)
        lp, tok = torch.topk(z, case["k"], dim=1)
        return dict(h=eh, lse=lse, lp=lp - lse[:, None], tok=tok)
    if case["N"] * case["k"] * case["V"] * _mean_len(case) > 3e10:
        return None   # takes too long
    return _search64(case, seed)


def _search64(case, seed):
    """The search itself in 64 bits, all inputs side by side (an input's
    outputs do not depend on the others)."""
    W, (h0, Lx, ml) = _inputs(case, seed)
    N, k, d, V, cap = case["N"], case["k"], case["d"], case["V"], _cap(case)
    fixed = case["sched"] == "fixed_stream"
    delta, M = (math.inf, k) if fixed else (case["delta"], case["M"])
    Wd = tuple(w.double() for w in W[:3])
    W_kv = None if W[3] is None else W[3].double()
    lx, ml = torch.from_numpy(Lx).cuda().double(), torch.from_numpy(ml).cuda()
    neg = -math.inf
    score = torch.full((N, k), neg, dtype=torch.float64, device="cuda")
    score[:, 0] = 0
    status = torch.zeros(N, k, dtype=torch.long, device="cuda")   # 0 empty, 1 active, 2 EOS, 3 cut
    status[:, 0] = 1
    h = torch.zeros(N, k, d, dtype=torch.float64, device="cuda")
    h[:, 0] = h0.double()
    last = torch.zeros(N, k, dtype=torch.long, device="cuda")
    toks = torch.zeros(N, k, cap, dtype=torch.int32, device="cuda")
    length = torch.zeros(N, k, dtype=torch.long, device="cuda")
    hist = None if not case["attn"] else torch.zeros(N, k, cap, 2 * case["kv"], d, dtype=torch.bfloat16, device="cuda")
    ranks = torch.arange(k, device="cuda")
    for t in range(1, cap + 1):
        live = torch.nonzero((status == 1).any(1)).flatten()
        if not len(live):
            break
        i, p = torch.nonzero(status[live] == 1, as_tuple=True)
        rows = live[i]
        x_of = None
        if hist is not None:
            def x_of(hs):
                for pl in range(2 * case["kv"]):
                    hist[rows, p, t - 1, pl] = _bf16(hs @ W_kv[pl // 2, pl % 2]).to(torch.bfloat16)
                out = torch.zeros_like(hs)
                for l in range(case["kv"]):
                    K = hist[rows, p, :t, 2 * l].double()
                    w = torch.softmax((K * hs[:, None, :]).sum(2) / math.sqrt(d), 1)
                    out += (w[:, :, None] * hist[rows, p, :t, 2 * l + 1].double()).sum(1)
                return _bf16(hs + out / case["kv"])
        _, hs, lse, z = _step64(case, Wd, h[rows, p], last[rows, p], case["beta"] * (t - lx[rows]), x_of)
        v, tk = torch.topk(z, k, dim=1)
        n = len(live)
        cs = torch.full((n, k, k + 1), neg, dtype=torch.float64, device="cuda")
        ct = torch.full((n, k, k + 1), -1, dtype=torch.long, device="cuda")
        cs[i, p, :k] = score[rows, p][:, None] + v - lse[:, None]
        ct[i, p, :k] = tk
        st = status[live]
        cs[:, :, k] = torch.where(st >= 2, score[live], neg)
        best, at = torch.sort(cs.reshape(n, -1), dim=1, descending=True, stable=True)
        best, at = best[:, :k], at[:, :k]
        par, tok = at // (k + 1), torch.gather(ct.reshape(n, -1), 1, at)
        ok = (best > neg) & (best >= best[:, :1] - delta)
        same = (par[:, :, None] == par[:, None, :]) & ok[:, None, :] & (tok[:, None, :] >= 0)
        before = (same & (ranks[None, :] < ranks[:, None])[None]).sum(2)
        ok &= (tok < 0) | (before < M)
        ns = torch.where(tok == 0, 2, torch.where(t == ml[live][:, None], 3, 1))
        ns = torch.where(tok < 0, torch.gather(st, 1, par), ns)
        ns = torch.where(ok, ns, 0)
        order = torch.sort(ok.to(torch.int8), dim=1, descending=True, stable=True)[1]
        best, par, tok, ns = (torch.gather(a, 1, order) for a in (best, par, tok, ns))
        new_h = h.clone()
        new_h[rows, p] = hs
        L = live[:, None]
        h[live] = new_h[L, par]
        if hist is not None:
            hist[live, :, :t] = hist[L, par, :t]
        old_tok, old_len = toks[L, par], length[L, par]
        g, r = torch.nonzero(tok >= 0, as_tuple=True)
        old_tok[g, r, old_len[g, r]] = tok[g, r].to(torch.int32)
        old_len[g, r] += 1
        toks[live], length[live] = old_tok, old_len
        last[live] = torch.where(tok >= 0, tok, torch.gather(last[live], 1, par))
        score[live], status[live] = torch.where(ns > 0, best, neg), ns
    count = (status > 0).sum(1)
    s = torch.gather(score, 1, torch.minimum(ranks[None, :], count[:, None] - 1))
    gone = status == 0
    length[gone] = 0
    toks[gone] = 0
    return dict(score=s, length=length.int(), status=status.int(), tokens=toks)
