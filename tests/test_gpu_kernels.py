"""Decoder-step kernels (recurrence, projection + log-sum-exp + per-row
top-k, row merge) against the oracle's fp64 decoder on explicit rows."""
import dataclasses

import numpy as np
import pytest

from oracle.decoder import ElmanDecoder
from synthgen import make_workload, scaled

pytestmark = pytest.mark.gpu


def _expand_case(wl, R, seed, h_prev=None):
    import torch
    from paper_2010_02164_amd import decoder_for_workload
    rng = np.random.default_rng(seed)
    c = wl.cfg
    dec = decoder_for_workload(wl, max_inputs=4)
    R = min(R, c.n * c.k)
    if h_prev is None:
        h_prev = np.tanh(rng.standard_normal((R, c.d))).astype(np.float32)
    R = h_prev.shape[0]
    if wl.is_bf16:
        from synthgen.gen import bf16_bits_to_f32, f32_to_bf16_bits
        h_prev = bf16_bits_to_f32(f32_to_bf16_bits(h_prev))
    y = rng.integers(0, c.V, R).astype(np.int32)
    t = rng.integers(1, 40, R).astype(np.int32)
    Lx = rng.integers(3, 40, R).astype(np.int32)
    hp = torch.from_numpy(h_prev).cuda()
    if wl.is_bf16:
        hp = hp.to(torch.bfloat16)
    h_gpu, lse, lp, tok = dec.debug_expand(hp, y, t, Lx)
    h_gpu = h_gpu.float().cpu().numpy()
    dec.close()
    o = ElmanDecoder.from_workload(wl)
    h_ref, lp_ref = o.expand(h_prev.astype(np.float64), y, t, Lx)
    z_ref = None
    return h_prev, y, t, Lx, h_gpu, lse, lp, tok, h_ref, lp_ref


def _check_rows(wl, h_gpu, lp, tok, h_ref, lp_ref, lse):
    k = wl.cfg.k
    if wl.is_bf16:
        assert np.array_equal(h_gpu, h_ref.astype(np.float32)), "bf16 states must be bit-identical"
    else:
        # fp32 accumulation over d products: the rounding error grows like
        # sqrt(d) * 2^-24 * |pre-activation| (|pre| <~ 4), ~8e-6 at d = 1024;
        # the bound allows 8 times that (6.1e-5 at d = 1024).
        tol = 8 * np.sqrt(wl.cfg.d) * 2.0**-24 * 4
        assert np.max(np.abs(h_gpu - h_ref)) < tol
    R = lp.shape[0]
    # log-sum-exp consistency: lp_ref of the GPU's tokens vs the GPU's lp
    for r in range(R):
        ref_row = lp_ref[r]
        kth = np.sort(ref_row)[::-1][:k]
        got = ref_row[tok[r]]
        assert np.all(np.abs(lp[r] - got) < 2e-5), (r, lp[r], got)
        # the GPU's list is a valid top-k: same values as the oracle's best k
        assert np.all(np.abs(np.sort(got)[::-1] - kth) < 2e-5)
        assert np.all(np.diff(lp[r]) <= 1e-12)          # best first
        assert len(set(tok[r].tolist())) == k


@pytest.mark.parametrize("cfg_i,R,over", [
    (1, 32, {}),                                   # V=1000 (ragged last tile), d=64
    (2, 300, {}),                                  # V=256, d=256, R not a tile multiple
    (3, 640, dict(V=8000)),                        # d=1024, k=5
    (1, 7, dict(V=130, k=3, M=3, n=4)),            # tiny ragged vocab, k < 4
])
def test_expand_f32(gpu, cfg_i, R, over):
    wl = make_workload(scaled(cfg_i, N=4, **over))
    _, _, _, _, h_gpu, lse, lp, tok, h_ref, lp_ref = _expand_case(wl, R, 11)
    print(f"[expand] cfg{cfg_i} {over} R={R}", flush=True)
    _check_rows(wl, h_gpu, lp, tok, h_ref, lp_ref, lse)


@pytest.mark.parametrize("over", [dict(V=8000, n=32), dict(V=4160, d=256, n=16, k=16),
                                  dict(V=32000, n=64), dict(V=32128, d=256, n=64)])
def test_expand_bf16(gpu, over):
    # The last two fill several rounds of tiles of 4 row blocks, over an even
    # and an odd number of vocabulary tiles.
    wl = make_workload(scaled(4, N=4, **over))
    _, _, _, _, h_gpu, lse, lp, tok, h_ref, lp_ref = _expand_case(wl, 640 if over["V"] >= 32000 else 200, 12)
    print(f"[expand] bf16 {over}", flush=True)
    _check_rows(wl, h_gpu, lp, tok, h_ref, lp_ref, lse)


# The bf16 recurrence sums W_h h exactly from 7-bit digits of the values
# scaled per W_h row and per state row, with the values too small for a
# row's 21-bit window added from per-row lists (a state row whose list
# overflows is scanned, a W_h whose lists overflow keeps the fp64 MFMA sum).
# These cases put such values, zeros, signed zeros, subnormals and large
# entries into W_h and the states; the states must stay bit-identical.
def _bf16(x):
    from synthgen.gen import bf16_bits_to_f32, f32_to_bf16_bits
    return bf16_bits_to_f32(f32_to_bf16_bits(np.asarray(x, np.float32)))


def _tiny(rng, cnt, lo=-40, hi=-16):
    return rng.choice([-1.0, 1.0], cnt) * 2.0 ** rng.uniform(lo, hi, cnt)


def _planted_wh(wl, rng, long_row=0):
    d = wl.cfg.d
    W = wl.W_h.copy()
    for o, cnt in [(0, 1), (1, 5), (2, 12), (40, 3), (1000 % d, 8)]:
        W[o, rng.choice(d, cnt, replace=False)] = _tiny(rng, cnt)
    W[7, 3] = 0.9                      # a large entry widens the row's window
    W[8, :5] = 1e-39                   # bf16 subnormals
    W[9, 10:20] = 0.0
    W[9, 20] = -0.0
    if long_row:
        W[5, rng.choice(d, long_row, replace=False)] = _tiny(rng, long_row)
    return dataclasses.replace(wl, W_h=_bf16(W))


def _planted_states(wl, rng, R):
    d = wl.cfg.d
    h = np.tanh(rng.standard_normal((R, d)))
    for r, cnt in [(0, 3), (1, 40), (5, 15), (6, 16), (33, 2), (70, 100)]:
        h[r, rng.choice(d, cnt, replace=False)] = _tiny(rng, cnt, -30, -14)
    h[2] = 0.0
    h[3, 0] = 6.0
    h[4, :8] = 1e-39 * np.sign(rng.standard_normal(8))
    h[4, 8:12] = -0.0
    h[7] = _tiny(rng, d, -30, -20)     # a row of small values only
    h[64:96] = 0.0                     # a whole tile of zero states
    if R > 1000:
        for r, cnt in [(700, 5), (701, 30), (1090, 15), (1099, 16)]:
            h[r, rng.choice(d, cnt, replace=False)] = _tiny(rng, cnt, -30, -14)
        h[1024:1088] = 0.0             # a whole 64-row tile of zero states
    return _bf16(h)


@pytest.mark.parametrize("long_row,R", [(0, 200), (40, 200), (0, 1100)])
def test_expand_bf16_small_values(gpu, long_row, R):
    # 1 100 rows run the 64 x 64 tiles (a step whose 64-row tiles fill half
    # the grid), 200 the 32 x 32 tiles with the K range split over waves.
    wl = _planted_wh(make_workload(scaled(4, N=4, V=8000, n=128)), np.random.default_rng(21), long_row)
    h_prev = _planted_states(wl, np.random.default_rng(22), R)
    _, _, _, _, h_gpu, lse, lp, tok, h_ref, lp_ref = _expand_case(wl, R, 23, h_prev=h_prev)
    print(f"[expand] bf16 small values long_row={long_row} R={R}", flush=True)
    _check_rows(wl, h_gpu, lp, tok, h_ref, lp_ref, lse)


@pytest.mark.parametrize("long_row", [0, 40])
def test_decode_bf16_small_values(gpu, long_row):
    """Whole decodes with encodings holding small values, zeros and large
    entries (their digits are made at submission) and the planted W_h (with
    a 40-value row list: the whole decode on the fp64 recurrence)."""
    from tests.gpu_util import check_parity
    rng = np.random.default_rng(31)
    wl = _planted_wh(make_workload(scaled(4, N=24, V=8000, n=8)), rng, long_row)
    h0 = wl.h0.copy()
    for i, cnt in [(0, 3), (1, 40), (2, 15), (3, 16)]:
        h0[i, rng.choice(wl.cfg.d, cnt, replace=False)] = _tiny(rng, cnt, -30, -12)
    h0[4] = 0.0
    h0[5, 0] = 60.0
    h0[6, :8] = 1e-39
    wl = dataclasses.replace(wl, h0=_bf16(h0))
    print(f"[parity] bf16 small values long_row={long_row}", flush=True)
    check_parity(wl, "var_stream")


# The fp32 projection splits W_out rows and states into fp16 pairs after a
# power-of-two scaling per W_out row. Large rows and an outlier inside a row keep
# each returned logit within a few units of 2^-24 of its products' sum of
# magnitudes (rows smaller than the others, which these outrank:
# test_expand_f32_wide_rows).
@pytest.mark.parametrize("V,d,R,k", [(130, 64, 1, 4), (1000, 192, 33, 12), (8320, 320, 97, 5), (32000, 64, 161, 8)])
def test_expand_f32_row_scales(gpu, V, d, R, k):
    rng = np.random.default_rng(41)
    wl = make_workload(scaled(1, N=4, V=V, d=d, k=k, M=k, n=-(-R // k)))
    W = wl.W_out.copy()
    W[1] *= 2.0**12
    W[5, d // 2] = 700.0
    W[V - 1] *= 2.0**8
    W[6:64] *= 2.0 ** rng.integers(-8, 6, 58)[:, None]
    W = W.astype(np.float32)
    wl = dataclasses.replace(wl, W_out=W)
    _, _, t, Lx, h_gpu, lse, lp, tok, _, _ = _expand_case(wl, R, 42)
    print(f"[expand] f32 row scales V={V} d={d} R={R}", flush=True)
    # Against the logits of the states that the step returned. Per logit: 6
    # units (WIDE_ROWS, below) and, for EOS, the bias' rounding; the log-sum-exp
    # is off by the logits' errors, weighted by their probabilities, plus its own
    # fp32 sum over |V| terms.
    h, Wd = h_gpu.astype(np.float64), W.astype(np.float64)
    z = h @ Wd.T
    z[:, 0] += wl.cfg.beta * (t - Lx)
    err = 6 * 2.0**-24 * (np.abs(h) @ np.abs(Wd).T)
    # One product makes up row 5's sum from the middle on: its d / 2 later
    # additions round by up to half a unit of it each (0.3 rms, times 4).
    err[:, 5] *= 1 + 1.2 * np.sqrt(d / 2) / 6
    err[:, 0] += 2.0**-24 * np.abs(z[:, 0])
    m = z.max(1, keepdims=True)
    ref_lse = m[:, 0] + np.log(np.exp(z - m).sum(1))
    lse_err = (np.exp(z - ref_lse[:, None]) * err).sum(1) + 1e-5
    assert np.all(np.abs(lse - ref_lse) < lse_err)
    assert np.all(np.abs(lp + lse[:, None] - np.take_along_axis(z, tok, 1)) <= np.take_along_axis(err, tok, 1) + 1e-12)
    assert np.all(np.diff(lp, axis=1) <= 1e-12)
    # No token left out is above one returned by more than their errors.
    low = np.take_along_axis(z + err, tok, 1).min(1)
    rest = z - err
    np.put_along_axis(rest, tok, -np.inf, 1)
    assert np.all(rest.max(1) <= low)


@pytest.mark.parametrize("V,d", [(1000, 64), (8320, 192)])
def test_expand_f32_infinite_weight(gpu, V, d):
    """An infinite W_out value whose product is -inf takes its token out of the
    row's sum and list and changes nothing else (one row: the sign of the
    state's value there decides); its neighbours have states whose low parts
    are zero, as a state of +-1 does."""
    wl = make_workload(scaled(1, N=4, V=V, d=d, k=5, M=5, n=1))
    E = wl.E.copy()
    E[:, d // 2] = 40.0   # tanh gives 1 exactly
    wl = dataclasses.replace(wl, E=E)
    _, _, _, _, _, _, _, tok0, h_ref, _ = _expand_case(wl, 1, 81)
    W = wl.W_out.copy()
    banned = [int(tok0[0, 0]), V - 1]
    for v, i in zip(banned, (3, d // 2)):
        W[v, i] = -np.inf * np.sign(h_ref[0, i])
    wl = dataclasses.replace(wl, W_out=W)
    _, _, _, _, _, lse, lp, tok, h_ref, lp_ref = _expand_case(wl, 1, 81)
    print(f"[expand] f32 infinite weight V={V} d={d}", flush=True)
    assert np.isneginf(lp_ref[0, banned]).all() and not set(banned) & set(tok[0].tolist())
    assert np.isfinite(lse).all() and np.abs(lp - np.take_along_axis(lp_ref, tok, 1)).max() < 1e-4
    assert np.array_equal(tok[0], np.argsort(-lp_ref[0], kind="stable")[:5])


@pytest.mark.parametrize("cfg_i,R", [(c, R) for c in (1, 4) for R in (1, 33, 65, 97, 129, 257)])
def test_expand_tile_heights(gpu, cfg_i, R):
    """Row tiles of 1 to 4 blocks with a ragged last block, in both types."""
    wl = make_workload(scaled(cfg_i, N=4, V=8320, d=128, k=5, M=4, n=52))
    _, _, _, _, h_gpu, lse, lp, tok, h_ref, lp_ref = _expand_case(wl, R, 51)
    print(f"[expand] {wl.cfg.dtype} R={R}", flush=True)
    _check_rows(wl, h_gpu, lp, tok, h_ref, lp_ref, lse)


@pytest.mark.parametrize("cfg_i", [1, 4])
@pytest.mark.parametrize("form", ["unaligned", "in_place", "noalloc", "again", "host", "pinned"])
def test_expand_state_buffers(gpu, cfg_i, form):
    """The step reads and writes the caller's state buffers where it can
    (this GPU's memory, 16-byte aligned, not overlapping) and copies otherwise; a decoder that
    allocates nothing copies its small arrays too. Same bits in every form."""
    import ctypes
    import torch
    from paper_2010_02164_amd import _native as N, decoder_for_workload
    wl = make_workload(scaled(cfg_i, N=4, V=1000, d=256, k=4, M=4, n=12))
    R, d, k = 45, 256, 4
    rng = np.random.default_rng(61)
    dt = torch.bfloat16 if wl.is_bf16 else torch.float32
    h = torch.from_numpy(np.tanh(rng.standard_normal((R, d))).astype(np.float32)).cuda().to(dt)
    y, t, lx = (rng.integers(a, b, R).astype(np.int32) for a, b in ((0, 1000), (1, 40), (3, 40)))
    dec = decoder_for_workload(wl, max_inputs=4)
    want = dec.debug_expand(h, y, t, lx)
    if form == "unaligned":
        x = torch.empty(R * d + 1, dtype=dt, device="cuda")[1:].view(R, d)
        x.copy_(h)
        got = dec.debug_expand(x, y, t, lx)
    elif form == "in_place":
        x = h.clone()
        lse, lp, tok = np.empty(R), np.empty((R, k)), np.empty((R, k), np.int32)
        I, D = ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_double)
        s = N.lib().sb_debug_expand(dec.handle, R, x.data_ptr(), y.ctypes.data_as(I), t.ctypes.data_as(I),
                                    lx.ctypes.data_as(I), x.data_ptr(), lse.ctypes.data_as(D), lp.ctypes.data_as(D),
                                    tok.ctypes.data_as(I))
        assert s == N.SB_OK
        got = (x, lse, lp, tok)
    elif form in ("host", "pinned"):
        x = h.cpu()
        got = dec.debug_expand(x.pin_memory() if form == "pinned" else x, y, t, lx)
        got = (got[0].cuda(),) + got[1:]
    elif form == "noalloc":
        nd = decoder_for_workload(wl, max_inputs=4, noalloc=True)
        got = nd.debug_expand(h, y, t, lx)
        nd.close()
    else:   # fewer rows, then the same again through the kept staging
        dec.debug_expand(h[:7], y[:7], t[:7], lx[:7])
        got = dec.debug_expand(h, y, t, lx)
    dec.close()
    assert torch.equal(got[0], want[0])
    for g, w in zip(got[1:], want[1:]):
        assert np.array_equal(g, w)


@pytest.mark.parametrize("cfg_i,k,per_tile", [(4, 16, 3), (1, 16, 3), (4, 9, 3), (1, 12, 4)])
def test_expand_one_lane_holds_the_best(gpu, cfg_i, k, per_tile):
    """Tiles t, t + 64, t + 128, t + 192 are merged by one lane, which keeps 8
    keys; here they hold 12 or 16 of a row's best tokens (with 4 in a tile the
    tile's short list may hide more as well)."""
    wl = make_workload(scaled(cfg_i, N=4, V=32000, d=128, k=k, M=4, n=4))
    rng = np.random.default_rng(71)
    u = rng.choice([-1.0, 1.0], 128)
    E = wl.E * 0.1 + 0.5 * u
    W = wl.W_out.copy()
    toks = [128 * (5 + 64 * i) + 7 * j + 3 for i in range(4) for j in range(per_tile)]
    for x, v in enumerate(toks):
        W[v] = u * (0.05 + 0.002 * ((5 * x) % len(toks)))
    cast = _bf16 if wl.is_bf16 else (lambda a: a.astype(np.float32))
    wl = dataclasses.replace(wl, E=cast(E), W_out=cast(W))
    _, _, _, _, h_gpu, lse, lp, tok, h_ref, lp_ref = _expand_case(wl, 37, 72)
    print(f"[expand] one lane {wl.cfg.dtype} k={k}", flush=True)
    assert len(set(tok[0].tolist()) & set(toks)) >= min(k, len(toks)) - 1
    _check_rows(wl, h_gpu, lp, tok, h_ref, lp_ref, lse)


# Logits of chosen tokens to their last bits. All tokens but 16 are held 50
# below, by a unit that is on (h = 1) in every row, and the first of the 16 has
# a row of zeros: its logit is 0, and the returned log-probabilities' differences
# to its own are the logits of the other 15. They are compared with 64-bit
# products of W_out and the states the step returned, as a multiple of 2^-24 of
# the products' sum of magnitudes.
ON, OFF, FAINT = 3, 7, 11   # units that are 1, 0 and 2^-27 in every row


def _logit_case(V, d, R, make, one_tile, seed=91, states=None):
    """(logits [R, 15], 64-bit logits, sums of magnitudes): the 15 chosen rows
    are make(rng, dense rows [15, d]); all in one 128-token tile or spread. With
    `states`, E and W_h are what it makes of them."""
    rng = np.random.default_rng(seed)
    wl = make_workload(scaled(1, N=4, V=V, d=d, k=16, M=16, n=-(-R // 16)))
    E, Wh, W = wl.E.copy(), wl.W_h.copy(), wl.W_out.copy()
    if states:
        E, Wh = states(rng, E, Wh)
    for u, e in ((ON, 40.0), (OFF, 0.0), (FAINT, 2.0**-27)):
        Wh[u], E[:, u] = 0.0, e
    W[:, ON] = -50.0
    at = 128 * (V // 256) + 5 + (7 * np.arange(16) if one_tile else 0)
    toks = at if one_tile else (5 + (V // 16) * np.arange(16))
    rows = rng.standard_normal((15, d)) * d**-0.5
    rows[:, [ON, OFF, FAINT]] = 0.0
    W[toks[0]] = 0.0
    W[toks[1:]] = make(rng, rows).astype(np.float32)
    wl = dataclasses.replace(wl, E=E.astype(np.float32), W_h=Wh.astype(np.float32), W_out=W.astype(np.float32))
    _, _, _, _, h, _, lp, tok, _, _ = _expand_case(wl, R, seed)
    order = np.argsort(tok, axis=1)
    assert np.array_equal(np.take_along_axis(tok, order, 1), np.tile(np.sort(toks), (R, 1)))
    lp = np.take_along_axis(lp, order, 1)[:, np.argsort(np.argsort(toks))]
    z = lp[:, 1:] - lp[:, :1]
    w, h = wl.W_out[toks[1:]].astype(np.float64), h.astype(np.float64)
    return z, h @ w.T, np.abs(h) @ np.abs(w).T


def _set(cols, value):
    def make(rng, rows):
        rows[:, cols] = value if np.ndim(value) == 0 else np.asarray(value)[:, None]
        return rows
    return make


def _keep(n):
    def make(rng, rows):   # n non-zero values in a row
        out = np.zeros_like(rows)
        for r in range(15):
            c = rng.choice(np.arange(12, rows.shape[1]), n, replace=False)
            out[r, c] = rows[r, c]
        return out
    return make


def _octaves(lo, hi, some=None):
    def make(rng, rows):   # all values, or some of each row, over many powers of two
        f = 2.0 ** rng.uniform(lo, hi, rows.shape)
        for r in range(15 if some else 0):
            f[r, rng.permutation(rows.shape[1])[some:]] = 1.0
        return rows * f
    return make


def _mixed(rng, rows):   # a tiny row, a zero one, and ordinary ones
    rows = rows * 2.0 ** rng.integers(-8, 3, (15, 1))
    rows[0] *= 2.0**-30
    rows[1] = 0.0
    return rows


# Units of 2^-24: a sum of n products rounded once per product is off by at most
# n; of many products by about 2.2 at most over these samples on the fp32 MFMA,
# and by up to 3.8 from pairs of fp16 (2^-21.2 = 7 for a single product).
WIDE_ROWS = [
    ("plain", lambda rng, rows: rows, 6), ("scaled", lambda rng, rows: rows * 2.0 ** rng.integers(-15, 1, (15, 1)), 6),
    ("mixed", _mixed, 6), ("subnormal_rows", lambda rng, rows: 0 * rows + 1e-41, 6),
    ("mask_1e9", _set([OFF], -1e9), 6), ("mask_1e12", _set([OFF], -1e12), 6), ("mask_3e38", _set([OFF], -3e38), 6),
    ("two_masks_up", _set([OFF, FAINT], [2.0**(30 - i) for i in range(15)]), 6), ("faint", _set([FAINT], -2.0**30), 6),
    ("tiny_values", _octaves(-50, -40, 3), 6), ("octaves", _octaves(-90, 0), 6), ("subnormal", _octaves(-140, -135, 80), 6),
    ("one_term", _keep(1), 1), ("two_terms", _keep(2), 2), ("forty_terms", _keep(40), 6),
]


@pytest.mark.parametrize("V,d", [(1000, 64), (8320, 256), (8320, 1024)])
@pytest.mark.parametrize("name,make,units", WIDE_ROWS, ids=[c[0] for c in WIDE_ROWS])
def test_expand_f32_wide_rows(gpu, name, make, units, V, d):
    """W_out rows whose values span more than the fp16 pairs hold (a large finite
    mask on a unit that is off, values next to zero), or with few non-zero ones,
    give their logits as the fp32 MFMA did; the row merge's recomputation of a
    saturated tile gives the same bits as the projection."""
    got = []
    for one_tile in (False, True):
        z, ref, mag = _logit_case(V, d, 45, make, one_tile)
        err = np.abs(z - ref) / np.maximum(mag, 2.0**-20) * 2.0**24
        print(f"[expand] f32 {name} V={V} d={d} one_tile={one_tile}: {err.max():.2f} units", flush=True)
        # lp are doubles of up to 200: differences carry 2^-45 of their own
        assert np.all(np.abs(z - ref) <= units * 2.0**-24 * mag + 2.0**-44)
        got.append(z)
    assert np.abs(got[0] - got[1]).max() <= 2.0**-44


def _scaled_states(e):
    return lambda rng, E, Wh: (E * 2.0**e, Wh * 2.0**e)


def _tiny_units(rng, E, Wh):   # some units far below the others
    u = rng.choice(np.arange(12, E.shape[1]), 6, replace=False)
    E[:, u], Wh[u] = E[:, u] * 2.0**-40, 0.0
    return E, Wh


def _few_units(n):
    def make(rng, E, Wh):   # n units that are not 0, with the ones of every row
        off = rng.permutation(np.setdiff1d(np.arange(E.shape[1]), [ON, OFF, FAINT]))[n:]
        E[:, off], Wh[off] = 0.0, 0.0
        return E, Wh
    return make


SMALL_STATES = [("2^-20", _scaled_states(-20), 20, 6), ("2^-26", _scaled_states(-26), 26, 6),
                ("2^-34", _scaled_states(-34), 34, 6), ("2^-60", _scaled_states(-60), 60, 6),
                ("tiny_units", _tiny_units, 0, 6), ("one_unit", _few_units(1), 0, 1), ("two_units", _few_units(2), 0, 2)]


@pytest.mark.parametrize("V,d", [(1000, 64), (8320, 256), (8320, 1024)])
@pytest.mark.parametrize("name,states,up,units", SMALL_STATES, ids=[c[0] for c in SMALL_STATES])
def test_expand_f32_small_states(gpu, name, states, up, units, V, d):
    """States smaller than the fp16 pairs hold, or few that are not zero, give
    their logits as the fp32 MFMA did (W_out is scaled up by as much)."""
    got = []
    for one_tile in (False, True):
        z, ref, mag = _logit_case(V, d, 45, lambda rng, rows: rows * 2.0**up, one_tile, states=states)
        err = np.abs(z - ref) / mag * 2.0**24
        print(f"[expand] f32 states {name} V={V} d={d} one_tile={one_tile}: {err.max():.2f} units", flush=True)
        assert np.all(np.abs(z - ref) <= units * 2.0**-24 * mag + 2.0**-44)
        got.append(z)
    assert np.abs(got[0] - got[1]).max() <= 2.0**-44


@pytest.mark.parametrize("V,k,R,one_in", [(1000, 4, 70, 2), (8320, 12, 200, 2), (8320, 5, 333, 9), (1000, 16, 300, 1.2)])
def test_expand_f32_rows_of_both_kinds(gpu, V, k, R, one_in):
    """Rows that need the fp32 MFMA change no bit of the rows that share their
    step, whose results are those of a step without them."""
    import torch
    from paper_2010_02164_amd import decoder_for_workload
    d = 256
    wl = make_workload(scaled(1, N=4, V=V, d=d, k=k, M=k, n=-(-R // k)))
    E, Wh = wl.E.copy(), np.zeros_like(wl.W_h)
    E[1::2] *= np.float32(2.0**-33)      # states of odd tokens
    wl = dataclasses.replace(wl, E=E, W_h=Wh)
    rng = np.random.default_rng(95)
    y = rng.integers(0, V // 2, R).astype(np.int32) * 2 + (rng.random(R) < 1 / one_in).astype(np.int32)
    y[:40] &= ~1                         # a block of plain rows, then both kinds
    t = rng.integers(1, 40, R).astype(np.int32)
    h = torch.zeros(R, d, device="cuda")
    dec = decoder_for_workload(wl, max_inputs=4)
    print(f"[expand] f32 rows of both kinds V={V} R={R}", flush=True)
    h1, lse, lp, tok = dec.debug_expand(h, y, t, t)
    for part in (y & 1 == 0, y & 1 == 1):
        n = int(part.sum())
        h2, lse2, lp2, tok2 = dec.debug_expand(h[:n].contiguous(), y[part], t[part], t[part])
        assert torch.equal(h1[torch.from_numpy(part).cuda()], h2)
        assert np.array_equal(lse[part], lse2) and np.array_equal(lp[part], lp2) and np.array_equal(tok[part], tok2)
    dec.close()


@pytest.mark.parametrize("kind", ["plain", "far", "fp32"])
def test_expand_f32_rows_do_not_depend_on_the_step(gpu, kind):
    """A row's bits are the same in steps of every tile height and of more than
    one group of row tiles, on each of the projection's ways."""
    import torch
    from paper_2010_02164_amd import decoder_for_workload
    V, d, R, k = 8320, 1024, 700, 12
    wl = make_workload(scaled(1, N=4, V=V, d=d, k=k, M=k, n=-(-R // k)))
    W = wl.W_out.copy()
    if kind == "far":
        W[np.arange(V), np.arange(V) % d] = -2.0**40
    elif kind == "fp32":
        W[::128, 100:] = 0.0
    rng = np.random.default_rng(97)
    h = torch.from_numpy(np.tanh(rng.standard_normal((R, d))).astype(np.float32)).cuda()
    y, t = rng.integers(0, V, R).astype(np.int32), rng.integers(1, 40, R).astype(np.int32)
    dec = decoder_for_workload(dataclasses.replace(wl, W_out=W), max_inputs=4)
    print(f"[expand] f32 {kind} rows in steps of several sizes", flush=True)
    whole = dec.debug_expand(h, y, t, t)
    for n in (1, 33, 65, 97, 129, 385):
        for r0 in (0, R - n):
            part = dec.debug_expand(h[r0:r0 + n].contiguous(), y[r0:r0 + n], t[r0:r0 + n], t[r0:r0 + n])
            assert torch.equal(part[0], whole[0][r0:r0 + n])
            for a, b in zip(part[1:], whole[1:]):
                assert np.array_equal(a, b[r0:r0 + n]), (n, r0)
    dec.close()
