"""GPU parity of the softmax branch's fp32-accurate kernels (operands as sums of bf16 terms) at the edges of their key tiles:
0, 1, 63, 64, 65 and 129 softmax tokens per head, the last tokens among them, forwards and backwards, and value rows
beyond the range of fp16."""
import numpy as np
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs, make_grad_output
from oracle import nats_oracle_bwd as nbw

from gpu_util import TOL, host, oracle_fwd, rel_err, stored, to_dev

pytestmark = pytest.mark.gpu
COUNTS = (0, 1, 63, 64, 65, 129)


def _inputs(dtype, d, L=192):
    x = make_fwd_inputs(1, len(COUNTS), L, d, dtype, 0.1, seed=800 + d)
    rng = np.random.default_rng(d)
    x["mask"][:] = 0
    for h, n in enumerate(COUNTS):       # the sequence's last token is among them
        x["mask"][0, h, np.append(rng.permutation(L - 1)[:n - 1], L - 1) if n else []] = 1
    return x


@pytest.mark.parametrize("combine_mode", [0, 1, 2])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
def test_forward_at_the_edges_of_the_key_tiles(dtype, d, combine_mode):
    x = _inputs(dtype, d)
    x["V"] *= 2.0 ** 20                   # exact in bf16, far beyond fp16
    g = to_dev(x, dtype)
    r = nats.hybrid_attn_fwd_ex(*(g[k] for k in ("Q", "K", "V", "alpha", "beta", "mask")), 64, math=nb.NATS_MATH_FP32,
                                combine_mode=combine_mode, want=("O_nla", "lse"))
    ref = oracle_fwd(x, mode=combine_mode, want=("O_nla", "lse"))
    torch.cuda.synchronize()
    assert rel_err(host(r["O"]), ref["O"], stored(dtype)) <= TOL["f32"]
    assert rel_err(host(r["O_nla"]), ref["O_nla"]) <= 1e-5
    lse, seen = host(r["lse"]), np.isfinite(ref["lse"])
    assert np.array_equal(np.isfinite(lse), seen)
    assert np.max(np.abs(lse[seen] - ref["lse"][seen])) <= 1e-5


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
def test_backward_at_the_edges_of_the_key_tiles(dtype, d):
    x = _inputs(dtype, d)
    dO = make_grad_output(1, len(COUNTS), 192, d, dtype, seed=810)
    g = to_dev(x, dtype)
    r = nats.hybrid_attn_bwd(*(g[k] for k in ("Q", "K", "V", "alpha", "beta", "mask")), torch.from_numpy(dO).to(g["Q"].dtype).cuda(),
                             want=("g_nla",))
    ref = nbw.hybrid_bwd(x["Q"], x["K"], x["V"], x["alpha"], x["beta"], x["mask"], dO)
    torch.cuda.synchronize()
    for key in ("dQ", "dK", "dV", "g_nla"):
        assert rel_err(host(r[key]), ref[key]) <= 1e-4, key
