"""GPU parity of the fused attention core (mpx_attention_fwd / _bwd) against
the oracle's attention_fwd / attention_bwd, through the C ABI.

Bars (per element), from the rounding steps both sides share:
  S    |dS| <= ulp(S) + 2 hd 2^-24 (|Q||K|^T)          (float32 vs float64 sums)
  P    |dP| <= P scale (dS + sum_j P_j dS_j) 1.1 + 2^-18 P + ulp(P)
       (first-order softmax sensitivity, float32 softmax error, final rounding)
  O    ulp(O) + 2 T 2^-24 (|P||V|) + |P_gpu - P_oracle| |V|
The backward takes the GPU's P on both sides; dP, dV, dQ, dK follow the GEMM
bar, dS adds the propagated dP difference and its float32 evaluation error,
and dQ / dK add the propagated dS bound.
"""
import math

import numpy as np
import pytest

from oracle import ops
from oracle.numfmt import round_to
from oracle.policy import Policy
from tests.gpu_util import HAVE_GPU, assert_within, to_dev_half, to_host, ulp

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not HAVE_GPU, reason="no GPU")]

if HAVE_GPU:
    import torch
    from paper_2507_03312_amd import binding as mx

HD = 64
# (B, H, T): every key-block count NB = ceil(T / 32) from 1 to 8 with ragged
# and full last blocks, both sides of the 128-token switch of the backward
SHAPES = [(2, 2, 1), (2, 3, 5), (1, 2, 32), (2, 2, 33), (2, 3, 65), (1, 2, 97), (1, 2, 128),
          (1, 2, 129), (1, 2, 160), (1, 2, 161), (1, 1, 192), (2, 2, 197), (1, 1, 200),
          (1, 2, 224), (1, 1, 225), (1, 2, 256)]


def _s():
    return torch.cuda.current_stream().cuda_stream


def _empty(shape, fmt):
    return torch.zeros(*shape, dtype=torch.float16 if fmt == "f16" else torch.bfloat16, device="cuda")


def _inputs(B, T, H, fmt, seed):
    rng = np.random.default_rng(seed)
    d = H * HD
    qkv = round_to(rng.normal(0.0, 1.0, size=(B * T, 3 * d)), fmt)
    dout = round_to(rng.normal(0.0, 1.0, size=(B * T, d)), fmt)
    return qkv, dout


def _abs(a):
    return np.abs(np.asarray(a, np.float64))


def _run(B, T, H, fmt, seed=0):
    pol = Policy(fmt)
    dt = mx.DTYPES[fmt]
    qkv, dout = _inputs(B, T, H, fmt, seed)
    d = H * HD
    ldP = -(-T // 8) * 8
    tq, tdo = to_dev_half(qkv, fmt), to_dev_half(dout, fmt)
    tO, tP, tdq = _empty((B * T, d), fmt), _empty((B * H * T, ldP), fmt), _empty((B * T, 3 * d), fmt)
    tP.fill_(7.0)  # padding must be overwritten with 0
    mx.mpx_attention_fwd(tq.data_ptr(), tO.data_ptr(), tP.data_ptr(), B, T, H, HD, dt, _s())
    ws_n = mx.mpx_attention_bwd_workspace(B, T, H, HD)
    ws = torch.zeros(max(ws_n, 16), dtype=torch.uint8, device="cuda")
    mx.mpx_attention_bwd(tq.data_ptr(), tP.data_ptr(), tdo.data_ptr(), tdq.data_ptr(), B, T, H, HD,
                         dt, ws.data_ptr() if ws_n else None, ws_n, _s())
    torch.cuda.synchronize()
    return pol, qkv, dout, to_host(tO), to_host(tP).reshape(B, H, T, ldP), to_host(tdq)


def _check_fwd(pol, fmt, qkv, B, T, H, gO, gPfull):
    scale = 1.0 / math.sqrt(HD)
    O_or, (q, k, v, P_or, _) = ops.attention_fwd(pol, qkv, B, T, H, HD)
    assert np.all(gPfull[..., T:] == 0.0), "P padding columns must be 0"
    gP = gPfull[..., :T]
    kt = np.swapaxes(k, -1, -2)
    S_or = pol.R(pol.mm(q, kt))
    dS = ulp(S_or, fmt) + 2 * HD * 2.0 ** -24 * (_abs(q) @ _abs(kt))
    Pv = _abs(P_or)
    bP = Pv * scale * (dS + (Pv * dS).sum(-1, keepdims=True)) * 1.1 + Pv * 2.0 ** -18 + ulp(P_or, fmt)
    assert_within(gP, P_or, bP, "P")
    dPm = np.abs(gP.astype(np.float64) - np.asarray(P_or, np.float64))
    O4 = np.asarray(O_or).reshape(B, T, H, HD).transpose(0, 2, 1, 3)
    bO = ulp(O4, fmt) + 2 * T * 2.0 ** -24 * (_abs(gP) @ _abs(v)) + dPm @ _abs(v)
    gO4 = gO.reshape(B, T, H, HD).transpose(0, 2, 1, 3)
    assert_within(gO4, O4, bO, "O")
    return q, k, v, gP


def _check_bwd(pol, fmt, qkv, dout, B, T, H, gP, gdq):
    scale = 1.0 / math.sqrt(HD)
    q, k, v = ops.split_heads(qkv, B, T, H, HD)
    P = np.asarray(gP, np.float64)
    ref = ops.attention_bwd(pol, (q, k, v, P, scale), dout, B, T, H, HD)
    rq, rk, rv = ops.split_heads(ref, B, T, H, HD)
    gq, gk, gv = ops.split_heads(gdq, B, T, H, HD)
    do = np.asarray(dout).reshape(B, T, H, HD).transpose(0, 2, 1, 3)
    vt = np.swapaxes(v, -1, -2)
    dP = pol.R(pol.mm(do, vt))
    ddP = ulp(dP, fmt) + 2 * HD * 2.0 ** -24 * (_abs(do) @ _abs(vt))
    dPv = np.asarray(dP, np.float64)
    rs = (dPv * P).sum(-1, keepdims=True)
    dS = pol.R(scale * P * (dPv - rs))
    ddS = (scale * P * (ddP + (P * ddP).sum(-1, keepdims=True)) * 1.1
           + scale * P * (np.abs(dPv) + np.abs(rs)) * 2.0 ** -21 + ulp(dS, fmt))
    Pt = np.swapaxes(P, -1, -2)
    bv = ulp(rv, fmt) + 2 * T * 2.0 ** -24 * (_abs(Pt) @ _abs(do))
    assert_within(gv, rv, bv, "dV")
    bq = ulp(rq, fmt) + 2 * T * 2.0 ** -24 * (_abs(dS) @ _abs(k)) + ddS @ _abs(k)
    assert_within(gq, rq, bq, "dQ")
    dSt, ddSt = np.swapaxes(dS, -1, -2), np.swapaxes(ddS, -1, -2)
    bk = ulp(rk, fmt) + 2 * T * 2.0 ** -24 * (_abs(dSt) @ _abs(q)) + ddSt @ _abs(q)
    assert_within(gk, rk, bk, "dK")


@pytest.mark.parametrize("fmt", ["f16", "bf16"])
@pytest.mark.parametrize("bth", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_fused_attention(fmt, bth):
    B, H, T = bth
    pol, qkv, dout, gO, gPfull, gdq = _run(B, T, H, fmt, seed=T)
    _, _, _, gP = _check_fwd(pol, fmt, qkv, B, T, H, gO, gPfull)
    _check_bwd(pol, fmt, qkv, dout, B, T, H, gP, gdq)


@pytest.mark.parametrize("T", [8, 16, 17, 31, 48, 49, 64, 80, 81, 96, 112, 113, 120, 136, 145, 177, 209, 241])
def test_fused_attention_group_edges(T):
    """Lengths at the edges of the groups of 8 keys and steps of 16 rows that
    the kernels skip or do not keep past T."""
    pol, qkv, dout, gO, gPfull, gdq = _run(2, T, 3, "bf16", seed=T)
    _, _, _, gP = _check_fwd(pol, "bf16", qkv, 2, T, 3, gO, gPfull)
    _check_bwd(pol, "bf16", qkv, dout, 2, T, 3, gP, gdq)


@pytest.mark.parametrize("fmt,bth", [("bf16", (128, 6, 65)), ("f16", (256, 6, 65)), ("bf16", (64, 12, 197))],
                         ids=lambda s: str(s))
def test_fused_attention_full_size(fmt, bth):
    """The ViT-block, ViT-S and ViT-B attention shapes, every element checked."""
    B, H, T = bth
    pol, qkv, dout, gO, gPfull, gdq = _run(B, T, H, fmt, seed=3)
    _, _, _, gP = _check_fwd(pol, fmt, qkv, B, T, H, gO, gPfull)
    _check_bwd(pol, fmt, qkv, dout, B, T, H, gP, gdq)


def test_fused_attention_limits():
    t = _empty((64, 3 * 64), "bf16")
    with pytest.raises(mx.MPXError, match="implemented for"):
        mx.mpx_attention_fwd(t.data_ptr(), t.data_ptr(), t.data_ptr(), 1, 257, 1, 64, mx.MPX_BF16, _s())
    with pytest.raises(mx.MPXError, match="implemented for"):
        mx.mpx_attention_bwd(t.data_ptr(), t.data_ptr(), t.data_ptr(), t.data_ptr(), 1, 8, 1, 32,
                             mx.MPX_BF16, None, 0, _s())



def _run_fwd(qkv, B, T, H, fmt):
    tq = to_dev_half(qkv, fmt)
    tO, tP = _empty((B * T, H * HD), fmt), _empty((B * H * T, -(-T // 8) * 8), fmt)
    mx.mpx_attention_fwd(tq.data_ptr(), tO.data_ptr(), tP.data_ptr(), B, T, H, HD, mx.DTYPES[fmt], _s())
    return to_host(tO), to_host(tP).reshape(B, H, T, -1)


@pytest.mark.parametrize("T,keys", [(16, [3]), (64, range(32, 64)), (160, range(0, 32)), (160, range(128, 160)),
                                    (161, [160]), (192, [40]), (197, [196]), (197, range(192, 197)),
                                    (256, range(224, 256)), (256, [0, 4, 255])], ids=str)
def test_nan_scores_reach_the_whole_row(T, keys):
    """NaN keys (one, the last of a ragged block, a whole block) make every
    probability of every query NaN, as a softmax over the row does, so a
    row's finite entries never hide an overflow."""
    qkv, _ = _inputs(1, T, 2, "bf16", seed=T)
    qkv = np.array(qkv)
    qkv[list(keys), 2 * HD:4 * HD] = np.nan  # K of both heads
    gO, gP = _run_fwd(qkv, 1, T, 2, "bf16")
    assert np.all(np.isnan(gP[..., :T])) and np.all(gP[..., T:] == 0.0)
    assert np.all(np.isnan(gO))


@pytest.mark.parametrize("T,keys", [(64, range(0, 32)), (160, range(0, 32)), (160, range(128, 160)), (197, range(0, 64)),
                                    (197, range(192, 197)), (256, range(0, 224))], ids=str)
def test_overflowed_scores_are_zero_probabilities(T, keys):
    """Scores that overflow to -inf in half (whole blocks of keys, first or
    last) give probabilities of exactly 0 and leave the other keys' softmax as
    it is."""
    fmt, keys = "f16", list(keys)
    qkv, _ = _inputs(1, T, 1, fmt, seed=T)
    qkv = np.array(qkv)
    qkv[:, 0], qkv[:, HD] = 200.0, 0.0
    qkv[keys, HD] = -400.0  # 200 * -400 lies below the smallest half
    gO, gP = _run_fwd(qkv, 1, T, 1, fmt)
    pol = Policy(fmt)
    q, k, v = ops.split_heads(qkv, 1, T, 1, HD)
    kt = np.swapaxes(k, -1, -2)
    S = np.asarray(pol.R(pol.mm(q, kt)), np.float64)
    assert np.all(np.isneginf(S[..., keys]))
    e = np.exp((S - S.max(-1, keepdims=True)) / 8.0)
    P = e / e.sum(-1, keepdims=True)
    dS = np.where(np.isfinite(S), ulp(np.where(np.isfinite(S), S, 0.0), fmt) + 2 * HD * 2.0 ** -24 * (_abs(q) @ _abs(kt)), 0.0)
    bP = P / 8.0 * (dS + (P * dS).sum(-1, keepdims=True)) * 1.1 + P * 2.0 ** -18 + ulp(P, fmt)
    assert np.all(gP[..., keys] == 0.0)
    assert_within(gP[..., :T], P, bP, "P")
    assert np.all(np.isfinite(gO))


@pytest.mark.parametrize("bht", [(1300, 4, 9), (400, 6, 20), (220, 7, 40), (200, 4, 50), (130, 4, 65), (50, 6, 81)],
                         ids=lambda s: "x".join(map(str, s)))
def test_backward_of_large_grids(bht):
    """Grids past what the chip holds at a time (up to 80 tokens P and dS then
    take K's place in LDS): the same bits as the same entries in grids of one."""
    B, H, T = bht
    fmt, d, ldP = "bf16", H * HD, -(-T // 8) * 8
    gen = torch.Generator(device="cuda").manual_seed(T)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    qkv, dout, dt = rnd(B, T, 3 * d), rnd(B, T, d), mx.DTYPES[fmt]
    O, P, dq = _empty((B, T, d), fmt), _empty((B, H * T, ldP), fmt), _empty((B, T, 3 * d), fmt)

    def run(x, g, o, p, out, n):
        mx.mpx_attention_fwd(x.data_ptr(), o.data_ptr(), p.data_ptr(), n, T, H, HD, dt, _s())
        mx.mpx_attention_bwd(x.data_ptr(), p.data_ptr(), g.data_ptr(), out.data_ptr(), n, T, H, HD, dt, None, 0, _s())

    run(qkv, dout, O, P, dq, B)
    for i in (0, 1, B // 2, B - 1):
        one = _empty((T, d), fmt), _empty((H * T, ldP), fmt), _empty((T, 3 * d), fmt)
        run(qkv[i], dout[i], *one, 1)
        for got, want in zip((O[i], P[i], dq[i]), one):
            assert torch.equal(got, want)
