"""NaN, infinities and decays outside (0, 1] in the fp32 forward: what a token brings reaches its own row and later ones, as
in the recurrence, and no row before it, whatever else shares its chunk."""
import numpy as np
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_chunk_mask, make_fwd_inputs

from gpu_util import host, oracle_fwd, rel_err, to_dev

pytestmark = pytest.mark.gpu
NAMES = ("Q", "K", "V", "alpha", "beta", "mask")


def _run(x, routing=nb.NATS_ROUTE_TOKEN, dtype="f32", **kw):
    g = to_dev(x, dtype)
    r = nats.hybrid_attn_fwd_ex(*(g[k] for k in NAMES), 64, math=nb.NATS_MATH_FP32, routing=routing,
                                want=("O_la", "O_nla", "lse", "final_state"), **kw)
    torch.cuda.synchronize()
    return {k: host(v) for k, v in r.items()}


def _same(got, ref):
    """the same values where finite, and not finite in the same places"""
    seen = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), seen)
    if seen.any():
        assert np.max(np.abs(got[seen] - ref[seen])) <= 1e-5 * np.sqrt(np.mean(ref[seen] ** 2))


@pytest.mark.parametrize("routing", [nb.NATS_ROUTE_TOKEN, nb.NATS_ROUTE_CHUNK])
@pytest.mark.parametrize("what,value", [("V", np.nan), ("V", np.inf), ("K", np.nan), ("Q", np.nan), ("alpha", np.nan),
                                        ("beta", np.nan)])
@pytest.mark.parametrize("t", [100, 191])
def test_linear_branch_takes_it_from_its_token_on(what, value, t, routing):
    x = make_fwd_inputs(1, 3, 192, 64, "f32", 0.2, seed=500)
    kw = {}
    if routing == nb.NATS_ROUTE_CHUNK:
        x["mask"] = make_chunk_mask(1, 3, 3, 0.5, seed=3)
        kw = dict(chunk_routing=64)
    else:
        x["mask"][0, :, t] = 0       # a linear token
    clean = _run(x, routing)
    for key in ("Q", "K", "V"):
        x[key] = x[key].copy()
    x[what][(0, 1, t, 5) if what in ("Q", "K", "V") else (0, 1, t)] = value
    got = _run(x, routing)
    with np.errstate(all="ignore"):
        ref = oracle_fwd(x, want=("O_la", "S"), **kw)
    assert not np.isfinite(got["O_la"][0, 1, t:]).all()
    for key, want in (("O_la", "O_la"), ("final_state", "S")):
        _same(got[key][0, 1], ref[want][0, 1])
        for h in (0, 2):              # the other heads are not touched
            assert np.array_equal(got[key][0, h], clean[key][0, h])


def test_prompts_padded_with_whatever_memory_holds():
    """Rows up to the prompt's end do not depend on the linear tokens that fill its last chunk."""
    x = make_fwd_inputs(2, 2, 256, 128, "f32", 0.1, seed=510)
    x["mask"][:, :, 217:] = 0
    ref = _run(x)
    for key in ("Q", "K", "V", "alpha", "beta"):
        x[key] = x[key].copy()
        x[key][:, :, 217:] = np.nan
    got = _run(x)
    for key in ("O", "O_la", "O_nla"):
        assert rel_err(got[key][:, :, :217], ref[key][:, :, :217]) <= 1e-5, key


@pytest.mark.parametrize("linear_op", [nb.NATS_LINEAR_GDN, nb.NATS_LINEAR_GATED])
def test_softmax_tokens_bring_nothing_to_the_state(linear_op):
    x = make_fwd_inputs(1, 2, 128, 64, "f32", 0.1, seed=520)
    x["mask"][0, :, 70] = 1
    ref = _run(x, linear_op=linear_op)
    x["V"] = x["V"].copy()
    x["V"][0, :, 70, 3] = np.nan
    got = _run(x, linear_op=linear_op)
    for key in ("O_la", "final_state"):
        assert rel_err(got[key], ref[key]) <= 1e-5, key


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_negative_and_growing_decays(dtype):
    """nats.h: the fp32 path has no limit on alpha."""
    x = make_fwd_inputs(1, 2, 192, 64, dtype, 0.1, seed=530)
    rng = np.random.default_rng(1)
    x["alpha"] = np.where(rng.random(x["alpha"].shape) < 0.1, -x["alpha"], x["alpha"]).astype(np.float32)
    x["alpha"][0, 1, 40:50] = 1.3
    got, ref = _run(x, dtype=dtype), oracle_fwd(x, want=("O_la", "S"))
    assert rel_err(got["O_la"], ref["O_la"]) <= 1e-5
    assert rel_err(got["final_state"], ref["S"]) <= 1e-5


def test_inner_part_left_out():
    """routing per chunk with the inner part of a chunk left to the softmax branch: no output row shows what the last chunk
    wrote, the final state does"""
    x = make_fwd_inputs(1, 2, 128, 64, "f32", 0.1, seed=540)
    x["mask"] = np.zeros((1, 2, 2), np.uint8)
    kw = dict(routing=nb.NATS_ROUTE_CHUNK, inner_chunk=1)
    clean = _run(x, **kw)
    x["V"] = x["V"].copy()
    x["V"][0, 1, 127, 5] = np.nan
    got = _run(x, **kw)
    want = clean["final_state"][0, 1].copy()
    want[5] = np.nan
    _same(got["final_state"][0, 1], want)
    _same(got["O_la"][0, 1], clean["O_la"][0, 1])
    assert np.array_equal(got["final_state"][0, 0], clean["final_state"][0, 0])


@pytest.mark.parametrize("routing", [nb.NATS_ROUTE_TOKEN, nb.NATS_ROUTE_CHUNK])
@pytest.mark.parametrize("what,value", [("V", np.nan), ("V", np.inf), ("V", -np.inf), ("K", np.nan), ("Q", np.nan)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64)])
def test_softmax_branch_takes_it_from_its_token_on(dtype, d, what, value, routing):
    x = make_fwd_inputs(1, 3, 320, d, dtype, 0.2, seed=550)
    kw, t = {}, 212
    if routing == nb.NATS_ROUTE_CHUNK:
        x["mask"] = make_chunk_mask(1, 3, 5, 0.5, seed=4)
        x["mask"][0, 1] = (1, 0, 0, 1, 0)
        kw = dict(chunk_routing=64)
    else:
        x["mask"][0, :, t] = 1
    clean = _run(x, routing, dtype)
    x[what] = x[what].copy()
    x[what][0, 1, t, 5] = value
    got = _run(x, routing, dtype)
    with np.errstate(all="ignore"):
        ref = oracle_fwd(x, want=("O_nla", "lse"), **kw)
    assert not np.isfinite(got["O_nla"][0, 1, t:]).all()
    for key in ("O_nla", "lse"):
        _same(got[key][0, 1], ref[key][0, 1])
        assert np.array_equal(got[key][0, 0], clean[key][0, 0]) and np.array_equal(got[key][0, 2], clean[key][0, 2])
