"""Distances of the fp32 calls from 64-bit arithmetic, as relative 2-norms over random inputs of the workloads' distributions:
the bars are what fp32 multiply-adds one after the other give, not a tolerance for any fp32 program."""
import numpy as np
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb

pytestmark = pytest.mark.gpu


def _inputs(B, H, L, d, p, seed):
    gen = torch.Generator().manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    unit = lambda *s: torch.nn.functional.normalize(rnd(*s), dim=-1)
    x = dict(Q=unit(B, H, L, d), K=unit(B, H, L, d), V=rnd(B, H, L, d), alpha=torch.sigmoid(2 + 0.5 * rnd(B, H, L)),
             beta=torch.sigmoid(rnd(B, H, L)), mask=(torch.rand(B, H, L, generator=gen) < p).to(torch.uint8))
    return {k: v.cuda() for k, v in x.items()}


def _recurrence(x):
    """O_la [B,H,L,d] and the last state of Eq. 19 / 20, in 64 bits."""
    q, k, v, a, b = (x[n].double() for n in ("Q", "K", "V", "alpha", "beta"))
    b = b * (x["mask"] == 0)
    B, H, L, d = q.shape
    S = torch.zeros(B, H, d, d, dtype=torch.float64, device=q.device)
    o = []
    for t in range(L):
        S = a[:, :, t, None, None] * S
        S = S + (b[:, :, t, None] * (v[:, :, t] - (S @ k[:, :, t, :, None])[..., 0]))[..., None] * k[:, :, t, None, :]
        o.append((S @ q[:, :, t, :, None])[..., 0])
    return torch.stack(o, 2), S


def _distance(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("d", [64, 128])
def test_linear_branch(d):
    x = _inputs(2, 3, 512, d, 0.1, seed=40 + d)
    got = nats.hybrid_attn_fwd_ex(*(x[n] for n in ("Q", "K", "V", "alpha", "beta", "mask")), 64, want=("O_la", "final_state"))
    o_la, state = _recurrence(x)
    # token by token, in fp32 multiply-adds, 7.0e-8 .. 8.5e-8; with a bias in the products 1.1e-7
    assert _distance(got["final_state"], state) <= 9.5e-8
    # token by token 1.0e-7 .. 1.1e-7; by chunks with q . k as one running sum 1.8e-7 .. 2.2e-7
    assert _distance(got["O_la"], o_la) <= 1.3e-7


@pytest.mark.parametrize("d", [64, 128])
def test_logits_of_one_sign(d):
    """Every query sees the first token alone, so lse is its logit; all numbers positive, so nothing that a product leaves
    out averages away."""
    rng = np.random.default_rng(d)
    x = _inputs(1, 2, 64, d, 0.0, seed=50 + d)
    for n in ("Q", "K"):   # mantissas whose later bits are all ones: the largest remainders
        bits = 0x3f800000 | rng.integers(0, 128, x[n].shape) << 16 | 0xffff
        x[n] = torch.from_numpy(bits.astype(np.uint32).view(np.float32)).cuda()
    x["mask"][:, :, 0] = 1
    got = nats.hybrid_attn_fwd_ex(*(x[n] for n in ("Q", "K", "V", "alpha", "beta", "mask")), 64, want=("lse",))["lse"]
    ref = (x["Q"].double() * x["K"].double()[:, :, :1]).sum(-1) / d ** 0.5
    # d products added in fp32 and scaled: a few roundings of 2^-24
    assert float(((got.double() - ref) / ref).abs().max()) <= 3e-7


@pytest.mark.parametrize("d", [64, 128])
def test_softmax_branch_with_large_logits(d):
    """Queries and keys of RMS norm 2, logits of up to 20: what rounds at the logits' size, not at that of their differences,
    shows.  Every token is a softmax token, so dV is the branch's too."""
    B, H, L = 1, 4, 512
    x = _inputs(B, H, L, d, 1.1, seed=60 + d)
    gen = torch.Generator().manual_seed(d)
    rms = lambda t: 2 * t / t.pow(2).mean(-1, keepdim=True).sqrt()
    q, k = (rms(torch.randn(B, H, L, d, generator=gen)).cuda() for _ in range(2))
    dO = torch.randn(B, H, L, d, generator=gen).cuda()
    args = [x[n] for n in ("Q", "K", "V", "alpha", "beta", "mask")]
    got = nats.hybrid_attn_fwd_ex(*args, 64, Q_nla=q, K_nla=k, want=("O_nla", "lse"))
    got.update(nats.hybrid_attn_bwd(*args, dO, 64, Q_nla=q, K_nla=k, want=("g_nla",)))
    q, k, v, g = (t.double() for t in (q, k, x["V"], dO))
    s = (q @ k.transpose(2, 3).contiguous() / d ** 0.5).masked_fill(~torch.ones(L, L, dtype=torch.bool, device="cuda").tril(), float("-inf"))
    lse = torch.logsumexp(s, -1)
    p = torch.exp(s - lse[..., None])
    o = p @ v
    ds = p * (g @ v.transpose(2, 3).contiguous() - (g * o).sum(-1, keepdim=True))
    # fp32 multiply-adds and expf one after the other: 4.8e-7, 3.9e-8, 8.0e-7, 8.8e-7, 7.0e-7, 8.8e-7 at L 1024, d 128
    for key, ref, bar in (("O_nla", o, 5e-7), ("lse", lse, 6e-8), ("dQ_nla", ds @ k / d ** 0.5, 8e-7),
                          ("dK_nla", ds.transpose(2, 3).contiguous() @ q / d ** 0.5, 8.8e-7),
                          ("dV", p.transpose(2, 3).contiguous() @ g, 7e-7), ("g_nla", ds.sum(2), 8.8e-7)):
        assert _distance(got[key], ref) <= bar, key


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [64, 128])
def test_gradients_of_the_plain_sum(d, dtype):
    from oracle import nats_oracle_bwd as nbw
    x = _inputs(1, 3, 320, d, 0.1, seed=70 + d)
    for n in ("Q", "K", "V"):
        x[n] = x[n].to(dtype)
    dO = torch.randn(1, 3, 320, d, generator=torch.Generator().manual_seed(d)).to(dtype).cuda()
    args = [x[n] for n in ("Q", "K", "V", "alpha", "beta", "mask")]
    got = nats.hybrid_attn_bwd(*args, dO, 64)
    ref = nbw.hybrid_bwd(*(t.float().cpu().numpy() if t.is_floating_point() else t.cpu().numpy() for t in args), dO.float().cpu().numpy())
    # over 40 drawn calls, fp32 multiply-adds and fp32 matrix instructions: at most 3.2e-7, 3.7e-7, 3.8e-7, 7.0e-7, 4.0e-7
    for key, bar in (("dQ", 3.2e-7), ("dK", 3.7e-7), ("dV", 3.8e-7), ("dalpha", 7e-7), ("dbeta", 4e-7)):
        assert _distance(got[key].cpu(), torch.from_numpy(np.asarray(ref[key], np.float64))) <= bar, key
