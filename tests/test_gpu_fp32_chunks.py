"""GPU parity of the forward in fp32 arithmetic with the linear branch by chunks of 64 tokens: the smallest lengths,
decays down to exactly 0 (whose ratios the chunk form takes through logarithms), and the fall-back to the token-by-token
recurrence where the states of all chunks do not fit the caller's memory."""
import numpy as np
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_chunk_mask, make_fwd_inputs

from gpu_util import TOL, host, oracle_fwd, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("routing", ["token", "chunk"])
@pytest.mark.parametrize("L,d", [(64, 64), (64, 128), (192, 128), (320, 64)])
def test_fp32_chunks_with_decays_down_to_zero(L, d, routing):
    x = make_fwd_inputs(1, 3, L, d, "f32", 0.2, seed=700 + L + d)
    rng = np.random.default_rng(L)
    kind = rng.random(x["alpha"].shape)
    x["alpha"] = np.where(kind < 0.1, 0.0, np.where(kind < 0.3, 10.0 ** rng.uniform(-12, -2, kind.shape), x["alpha"]))
    x["alpha"] = x["alpha"].astype(np.float32)
    x["beta"] = np.where(kind > 0.9, 0.0, np.where(kind > 0.8, 1.0, x["beta"])).astype(np.float32)
    kw, okw = {}, {}
    if routing == "chunk":
        x["mask"] = make_chunk_mask(1, 3, L // 64, 0.5, seed=L)
        kw, okw = dict(routing=nb.NATS_ROUTE_CHUNK), dict(chunk_routing=64)
    g = to_dev(x, "f32")
    r = nats.hybrid_attn_fwd_ex(g["Q"], g["K"], g["V"], g["alpha"], g["beta"], g["mask"], 64,
                                want=("O_la", "final_state"), **kw)
    ref = oracle_fwd(x, want=("O_la", "S"), **okw)
    torch.cuda.synchronize()
    assert rel_err(host(r["O"]), ref["O"]) <= TOL["f32"]
    # every decay ratio to a few fp32 roundings: ten times tighter than the bar of the fp32 path
    assert rel_err(host(r["O_la"]), ref["O_la"]) <= 1e-5
    assert rel_err(host(r["final_state"]), ref["S"]) <= 1e-5


def test_noalloc_forward_falls_back_to_the_recurrence():
    B, H, L, d = 1, 1, 16384, 128       # 25 MB token by token, 51 MB with a state per chunk
    assert nb.fwd_workspace_bytes(nb.make_fwd_params(B, H, L, d, 64, nb.NATS_F32)) > nb.NOALLOC_SCRATCH_BYTES
    x = make_fwd_inputs(B, H, L, d, "f32", 0.02, seed=710)
    g = to_dev(x, "f32")
    out = nats.hybrid_attn_fwd_noalloc(*(g[k] for k in ("Q", "K", "V", "alpha", "beta", "mask")), torch.empty_like(g["Q"]))
    torch.cuda.synchronize()
    assert rel_err(host(out), oracle_fwd(x, want=())["O"]) <= TOL["f32"]
