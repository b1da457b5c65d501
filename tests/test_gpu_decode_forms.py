"""GPU parity of the generation step's forms at the edges of their parts: cache lengths around 64 and 256 rows (and 0), a
full cache, few and many (batch, head) pairs, with no workspace given, with one of the documented size and with a
larger one, for both routings; a step refused by the host path raises what the checks say."""
import numpy as np
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from oracle import c_oracle

from gpu_util import TOL, host, rel_err, stored

pytestmark = pytest.mark.gpu


def _state(B, H, d, cap, dtype, seed, lens_given=None):
    rng = np.random.default_rng(seed)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    rnd = lambda *s: torch.from_numpy(rng.standard_normal(s).astype(np.float32)).to(tdt).float().numpy()
    unit = lambda *s: torch.from_numpy((lambda x: x / np.linalg.norm(x, axis=-1, keepdims=True))(rng.standard_normal(s)).astype(np.float32)).to(tdt).float().numpy()
    lens = rng.choice(lens_given or [0, 1, 63, 64, 65, 255, 256, 257, cap - 1, cap], size=(B, H)).astype(np.int32)
    lens.flat[0] = cap if lens_given is None else lens_given[-1]
    x = dict(state=(0.02 * rng.standard_normal((B, H, d, d))).astype(np.float32), k_cache=unit(B, H, cap, d),
             v_cache=rnd(B, H, cap, d), cache_len=lens, q=unit(B, H, d), k=unit(B, H, d), v=rnd(B, H, d),
             alpha=rng.uniform(0.5, 1, (B, H)).astype(np.float32), beta=rng.uniform(0, 1, (B, H)).astype(np.float32),
             mask=(rng.random((B, H)) < 0.5).astype(np.uint8))
    g = {k: torch.from_numpy(v).cuda() for k, v in x.items()}
    for k in ("k_cache", "v_cache", "q", "k", "v"):
        g[k] = g[k].to(tdt)
    return x, g


FORMS = ("none", "exact", "large")


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("dtype,B,H,d", [("bf16", 1, 7, 128), ("bf16", 5, 8, 64), ("f32", 2, 3, 128), ("bf16", 18, 15, 64)])
def test_decode_step_in_every_form(dtype, B, H, d, form):
    cap = 330
    x, g = _state(B, H, d, cap, dtype, seed=900 + B)
    ws = None
    if form != "none":
        n = nb.decode_workspace_bytes(B, H, d, cap, nb.NATS_F32 if dtype == "f32" else nb.NATS_BF16)
        ws = torch.full((n * (1 if form == "exact" else 5),), 0xFF, dtype=torch.uint8, device="cuda")
    err = torch.full((B, H), 7, dtype=torch.int32, device="cuda")
    o = nats.hybrid_attn_decode(g["state"], g["k_cache"], g["v_cache"], g["cache_len"], *(g[k] for k in ("q", "k", "v", "alpha", "beta", "mask")),
                                err_flags=err, workspace=ws)
    torch.cuda.synchronize()
    st, kc, vc, ln = x["state"].astype(np.float64), x["k_cache"].copy(), x["v_cache"].copy(), x["cache_len"].copy()
    ref, over = c_oracle.decode(st, kc, vc, ln, x["q"], x["k"], x["v"], x["alpha"], x["beta"], x["mask"])
    assert rel_err(host(o), ref, stored(dtype)) <= TOL[dtype]
    assert rel_err(host(g["state"]), st) <= 1e-5
    assert np.array_equal(host(g["cache_len"]), ln) and np.array_equal(host(err) != 0, over != 0)
    assert np.array_equal(host(g["k_cache"]), kc) and np.array_equal(host(g["v_cache"]), vc)


@pytest.mark.parametrize("dtype,B,H,d", [("bf16", 1, 5, 128), ("f32", 2, 3, 128), ("bf16", 18, 15, 128), ("bf16", 3, 4, 64)])
def test_chunk_of_generation_in_every_form(dtype, B, H, d):
    """128 pairs and fewer with d = 128 run as blocks of equal size, the others as one block per pair."""
    cap, n = 330, 3
    x, g = _state(B, H, d, cap, dtype, seed=950 + B)
    st = dict(state=g["state"], state_start=torch.empty_like(g["state"]), chunk_decay=torch.ones((B, H), device="cuda"),
              chunk_pos=torch.zeros((B, H), dtype=torch.int32, device="cuda"), k_cache=g["k_cache"], v_cache=g["v_cache"],
              cache_len=g["cache_len"])
    S, kc, vc = x["state"].astype(np.float64), x["k_cache"].astype(np.float64), x["v_cache"].astype(np.float64)
    for t in range(n):
        o = host(nats.hybrid_attn_decode_chunk(st, g["q"], g["k"], g["v"], g["alpha"], g["beta"]))
        a, b = x["alpha"][..., None, None].astype(np.float64), x["beta"][..., None].astype(np.float64)
        S = a * S
        S = S + (b * (x["v"] - np.einsum("bhij,bhj->bhi", S, x["k"])))[..., None] * x["k"][..., None, :]
        ref = np.einsum("bhij,bhj->bhi", S, x["q"])
        for i in np.ndindex(B, H):
            row = x["cache_len"][i] + t
            if row < cap: kc[i][row], vc[i][row] = x["k"][i], x["v"][i]
            m = min(row + 1, cap)
            s = kc[i][:m] @ x["q"][i] / np.sqrt(d)
            p = np.exp(s - s.max())
            ref[i] += (p / p.sum()) @ vc[i][:m]
        assert rel_err(o, ref, stored(dtype)) <= TOL[dtype], t
    assert rel_err(host(g["state"]), S) <= 1e-5
    assert np.all(host(st["chunk_pos"]) == n) and np.array_equal(host(st["cache_len"]), x["cache_len"])
    assert np.allclose(host(st["chunk_decay"]), x["alpha"].astype(np.float64) ** n, rtol=1e-6)
    assert np.array_equal(host(st["state_start"]), x["state"])


# One block of sixteen wavefronts per (batch, head), which walks the cache by STEP rows with two sets of registers in turn: d 128
# with 129 .. 256 pairs, d 64 with a cache below 2048 rows; no workspace, or the step would run in parts.
WIDE = [("bf16", 9, 16, 128, 192), ("bf16", 1, 5, 64, 384), ("f32", 9, 16, 128, 96), ("f32", 2, 3, 64, 192)]
WIDE_IDS = ["wide_%s_d%d" % (c[0], c[3]) for c in WIDE]


@pytest.mark.parametrize("dtype,B,H,d,step", WIDE, ids=WIDE_IDS)
def test_long_walks_of_the_wide_block(dtype, B, H, d, step):
    cap = 3 * step + 24
    x, g = _state(B, H, d, cap, dtype, seed=970 + d, lens_given=[0, step - 1, step, step + 1, 2 * step, 2 * step + 1, 3 * step, cap])
    o = nats.hybrid_attn_decode(g["state"], g["k_cache"], g["v_cache"], g["cache_len"], *(g[k] for k in ("q", "k", "v", "alpha", "beta", "mask")))
    torch.cuda.synchronize()
    st, kc, vc, ln = x["state"].astype(np.float64), x["k_cache"].copy(), x["v_cache"].copy(), x["cache_len"].copy()
    ref, _ = c_oracle.decode(st, kc, vc, ln, x["q"], x["k"], x["v"], x["alpha"], x["beta"], x["mask"])
    assert rel_err(host(o), ref, stored(dtype)) <= TOL[dtype]
    assert rel_err(host(g["state"]), st) <= 1e-5
    assert np.array_equal(host(g["cache_len"]), ln)
    assert np.array_equal(host(g["k_cache"]), kc) and np.array_equal(host(g["v_cache"]), vc)


@pytest.mark.parametrize("dtype,B,H,d,step", WIDE, ids=WIDE_IDS)
def test_long_walks_of_the_wide_block_by_chunks(dtype, B, H, d, step):
    """The second token of an open chunk finds the first one's row behind the cache's length."""
    cap = 3 * step + 24
    x, g = _state(B, H, d, cap, dtype, seed=980 + d, lens_given=[0, step - 2, step - 1, step, 2 * step - 1, 2 * step, 3 * step - 1, 3 * step])
    st = dict(state=g["state"], state_start=torch.empty_like(g["state"]), chunk_decay=torch.ones((B, H), device="cuda"),
              chunk_pos=torch.zeros((B, H), dtype=torch.int32, device="cuda"), k_cache=g["k_cache"], v_cache=g["v_cache"],
              cache_len=g["cache_len"])
    S = x["state"].astype(np.float64)
    a, b = x["alpha"][..., None, None].astype(np.float64), x["beta"][..., None].astype(np.float64)
    kc, vc = x["k_cache"].astype(np.float64), x["v_cache"].astype(np.float64)
    for t in range(2):
        o = host(nats.hybrid_attn_decode_chunk(st, g["q"], g["k"], g["v"], g["alpha"], g["beta"]))
        S = a * S
        S = S + (b * (x["v"] - (S @ x["k"][..., None])[..., 0]))[..., None] * x["k"][..., None, :]
        ref = (S @ x["q"][..., None])[..., 0]
        for i in np.ndindex(B, H):
            n = x["cache_len"][i] + t + 1
            kc[i][n - 1], vc[i][n - 1] = x["k"][i], x["v"][i]
            z = kc[i][:n] @ x["q"][i] / np.sqrt(d)
            p = np.exp(z - z.max())
            ref[i] += (p / p.sum()) @ vc[i][:n]
        assert rel_err(o, ref, stored(dtype)) <= TOL[dtype], t
    assert rel_err(host(g["state"]), S) <= 1e-5


def test_refused_steps_say_why():
    _, g = _state(1, 2, 64, 96, "bf16", seed=1)
    a = [g[k] for k in ("state", "k_cache", "v_cache", "cache_len", "q", "k", "v", "alpha", "beta", "mask")]
    with pytest.raises(ValueError, match="alpha must be contiguous"):
        nats.hybrid_attn_decode(*a[:7], a[7].double(), *a[8:])
    with pytest.raises(ValueError, match="q must be a GPU tensor"):
        nats.hybrid_attn_decode(*a[:4], a[4].cpu(), *a[5:])
    with pytest.raises(nb.NatsError, match="combine_mode"):
        nats.hybrid_attn_decode(*a, combine_mode=9)
    with pytest.raises(nb.NatsError, match="workspace of 16 bytes"):
        nats.hybrid_attn_decode(*a, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
