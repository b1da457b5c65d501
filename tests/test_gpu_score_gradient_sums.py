"""Chunk score gradients of Eq. 16 against 64-bit arithmetic.  They are sums of dS = P (dP - D) over all queries of a head,
and over the rows that a query sees dS sums to zero: an error of one sign in dP adds up over the queries while the sum itself
does not grow.  (The bf16 matrix instruction truncates towards minus infinity as it accumulates, 1 part in 2^24 or so.)"""
import ctypes

import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb

from test_bwd_bf16_overlaps import EXTRA

pytestmark = pytest.mark.gpu
C = 64


def _exact(Q, K, V, dO, mask, G):
    """dscore_nla [B,H,L/C] of the plain sum, in 64 bits: the linear branch has no part in it."""
    rep = lambda t: t.double().repeat_interleave(G, 1)
    B, H, L, d = Q.shape
    q, k, v, g, m = rep(Q), rep(K), V.double(), dO.double(), mask.bool().repeat_interleave(G, 1)
    t = torch.arange(L, device=Q.device)
    before = t[:, None] // C > t[None] // C
    if mask.shape[2] == L:                                   # routing per token
        see = (t[:, None] >= t[None]) & m[:, :, None]
        own = torch.zeros_like(see)
    else:
        own = ((t[:, None] >= t[None]) & ~before).expand(B, H * G, L, L)
        see = before & m.repeat_interleave(C, 2)[:, :, None]
    s = (q @ k.transpose(2, 3).contiguous() / d ** 0.5).masked_fill(~(see | own), float("-inf"))
    p = torch.nan_to_num(torch.softmax(s, -1))
    dp = g @ v.transpose(2, 3).contiguous()
    ds = p * (dp - (p * dp).sum(-1, keepdim=True)) * see
    return ds.sum(2).view(B, H, G, L // C, C).sum((2, 4))


@pytest.mark.parametrize("routing", [nb.NATS_ROUTE_TOKEN, nb.NATS_ROUTE_CHUNK])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,H,G,L,d", [(2, 2, 2, 768, 128), (3, 4, 1, 704, 64), (2, 2, 1, 1664, 128)])
def test_distance_to_64_bits(B, H, G, L, d, dtype, routing):
    gen = torch.Generator().manual_seed(L + d)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    unit = lambda *s: torch.nn.functional.normalize(rnd(*s), dim=-1).to(dtype).cuda()
    Q, K, V, dO = unit(B, H, L, d), unit(B, H, L, d), rnd(B, H * G, L, d).to(dtype).cuda(), rnd(B, H * G, L, d).to(dtype).cuda()
    alpha, beta = torch.sigmoid(2 + 0.5 * rnd(B, H, L)).cuda(), torch.sigmoid(rnd(B, H, L)).cuda()
    n = L // C if routing == nb.NATS_ROUTE_CHUNK else L
    mask = (torch.rand(B, H, n, generator=gen) < 0.1).to(torch.uint8).cuda()
    mask[:, :, 0] = 1
    got = nats.hybrid_attn_bwd(Q, K, V, alpha, beta, mask, dO, C, routing=routing, group=G, want=("dscore_nla",))["dscore_nla"]
    ref = _exact(Q, K, V, dO, mask, G)
    # a dS is some ten fp32 roundings of 2^-24 of P dP, and a sum over queries and keys that cancels to a third of the
    # size its terms would give at random keeps that; measured 3e-7 .. 1.1e-6, with an error of one sign 2e-6 .. 8e-6
    assert float((got - ref).norm() / ref.norm()) <= 1.5e-6


@pytest.mark.parametrize("routing", [nb.NATS_ROUTE_TOKEN, nb.NATS_ROUTE_CHUNK])
@pytest.mark.parametrize("G", [1, 3])
def test_a_chunk_score_is_rounded_once(G, routing):
    """Eq. 16 and 17 as sums over a chunk of what the same call returns per token: one rounding, whatever cancels."""
    B, H, L, d = 2, 3, 320, 64
    gen = torch.Generator().manual_seed(7)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    unit = lambda: torch.nn.functional.normalize(rnd(B, H, L, d), dim=-1).cuda()
    beta = torch.sigmoid(rnd(B, H, L)).cuda()
    mask = (torch.rand(B, H, L // (C if routing else 1), generator=gen) < 0.3).to(torch.uint8).cuda()
    want = ("g_nla", "dscore_nla") + (() if routing else ("dscore_la",))
    r = nats.hybrid_attn_bwd(unit(), unit(), rnd(B, H * G, L, d).cuda(), torch.sigmoid(2 + rnd(B, H, L)).cuda(), beta, mask,
                             rnd(B, H * G, L, d).cuda(), C, routing=routing, group=G, want=want)
    sums = dict(dscore_nla=r["g_nla"].double())
    if not routing:
        sums["dscore_la"] = beta.double() * r["dbeta"].double() * (mask == 0)
    for key, per_token in sums.items():
        ref = per_token.view(B, H, L // C, C).sum(-1)
        assert bool(((r[key].double() - ref).abs() <= 2.0 ** -24 * 1.001 * ref.abs()).all()), key


@pytest.mark.parametrize("way", ["plain", "at_once", "members"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_chunks_of_128_tokens(dtype, way):
    """Routing per token, C = 128: L / 128 sums, and nothing behind them."""
    B, H, L, d, G = 2, 2, 384, 64, 1 if way == "plain" else 2
    gen = torch.Generator().manual_seed(9)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    unit = lambda: torch.nn.functional.normalize(rnd(B, H, L, d), dim=-1).to(dtype).cuda()
    x = dict(Q=unit(), K=unit(), V=rnd(B, H * G, L, d).to(dtype).cuda(), alpha=torch.sigmoid(2 + rnd(B, H, L)).cuda(),
             beta=torch.sigmoid(rnd(B, H, L)).cuda(), mask=(torch.rand(B, H, L, generator=gen) < 0.3).to(torch.uint8).cuda(),
             dO=rnd(B, H * G, L, d).to(dtype).cuda())
    n = B * H * L // 128
    out = {k: torch.full(s, 7.0, device="cuda") for k, s in dict(
        dQ=(B, H, L, d), dK=(B, H, L, d), dV=(B, H * G, L, d), dalpha=(B, H, L), dbeta=(B, H, L), g_nla=(B, H, L), g_la=(B, H, L),
        dscore_nla=(4 * n,), dscore_la=(4 * n,)).items()}
    lib = nb.load_library()
    p = nb.make_fwd_params(B, H, L, d, 128, nb.NATS_F32 if dtype == torch.float32 else nb.NATS_BF16, group=G)
    size = lib.nats_hybrid_attn_bwd_workspace_bytes(ctypes.byref(p)) * (2 if way == "at_once" else 1)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    ex = nb.BwdExtra(*(out[k].data_ptr() if k in out else None for k in EXTRA))
    a = [ctypes.c_void_p(t.data_ptr()) for t in (*x.values(), *list(out.values())[:5])]
    assert lib.nats_hybrid_attn_bwd(ctypes.byref(p), *a, ctypes.byref(ex), ctypes.c_void_p(ws.data_ptr()), size,
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()
    # dscore_la: sums of products of which g_la holds the rounded ones, half an ulp (2^-24) of each; a member's score is rounded
    # before it is added to the others'
    for key, g in (("dscore_nla", out["g_nla"]), ("dscore_la", out["g_la"])):
        assert bool((out[key][n:] == 7.0).all()), key
        terms = g.double().view(n, 128)
        bound = 2.0 ** -24 * (4 * terms.abs().sum(-1) + terms.sum(-1).abs())
        assert bool(((out[key][:n].double() - terms.sum(-1)).abs() <= bound).all()), key
