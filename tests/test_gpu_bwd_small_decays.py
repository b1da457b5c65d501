"""The backward pass by chunks with decays down to exactly 0, whose ratios and gradients go through logarithms."""
import numpy as np
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_chunk_mask, make_fwd_inputs, make_grad_output
from oracle import nats_oracle_bwd as nbw

from gpu_util import host, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("routing", [nb.NATS_ROUTE_TOKEN, nb.NATS_ROUTE_CHUNK])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
def test_decays_down_to_zero(dtype, d, routing):
    B, H, L = 1, 3, 192
    x = make_fwd_inputs(B, H, L, d, dtype, 0.2, seed=600 + d)
    rng = np.random.default_rng(d)
    kind = rng.random((B, H, L))
    x["alpha"] = np.where(kind < 0.1, 0.0, np.where(kind < 0.4, 10.0 ** rng.uniform(-12, -2, kind.shape), x["alpha"])).astype(np.float32)
    dO = make_grad_output(B, H, L, d, dtype, seed=610)
    if routing == nb.NATS_ROUTE_CHUNK:
        x["mask"] = make_chunk_mask(B, H, L // 64, 0.4, seed=5)
        with np.errstate(all="ignore"):      # its dalpha at 0
            ref = nbw.hybrid_bwd_chunk_routed(x["Q"], x["K"], x["V"], x["alpha"], x["beta"], x["mask"], 64, dO)
    else:
        ref = nbw.hybrid_bwd(x["Q"], x["K"], x["V"], x["alpha"], x["beta"], x["mask"], dO)
    g = to_dev(x, dtype)
    r = nats.hybrid_attn_bwd(*(g[k] for k in ("Q", "K", "V", "alpha", "beta", "mask")), torch.from_numpy(dO).to(g["Q"].dtype).cuda(),
                             routing=routing)
    torch.cuda.synchronize()
    for key in ("dQ", "dK", "dV", "dbeta"):
        assert rel_err(host(r[key]), ref[key]) <= 1e-5, key      # a ratio from floats of log2 gamma: 1e-4 and more
    da, zero = host(r["dalpha"]), x["alpha"] == 0
    assert np.isfinite(da).all() and (da[zero] == 0).all()
    # sums of fp32 terms, 2^-24 of the size of their largest, divided by alpha
    assert rel_err((da * x["alpha"])[~zero], (ref["dalpha"] * x["alpha"])[~zero]) <= 1e-5
