"""GPU parity of the linear branch's backward by chunks (products on bf16 terms) where its parts could go wrong: one, two,
three and five chunks (the operands' sets in flight take turns), beta exactly 0 and 1 (the residuals are kept without
that factor, dbeta comes from sums over a chunk), strong decay, and a state handed in."""
import numpy as np
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs, make_grad_output
from oracle import nats_oracle_bwd as nbw

from gpu_util import host, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("linear_op", [nb.NATS_LINEAR_GDN, nb.NATS_LINEAR_GATED])
@pytest.mark.parametrize("n_chunks", [1, 2, 3, 5])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
def test_chunks_and_gates(dtype, d, n_chunks, linear_op):
    B, H, L = 1, 2, 64 * n_chunks
    x = make_fwd_inputs(B, H, L, d, dtype, 0.2, seed=700 + d + n_chunks)
    rng = np.random.default_rng(n_chunks)
    x["beta"][rng.random((B, H, L)) < 0.2] = 0.0
    x["beta"][rng.random((B, H, L)) < 0.1] = 1.0
    x["alpha"][rng.random((B, H, L)) < 0.1] = 1e-3
    S0 = (0.1 * rng.standard_normal((B, H, d, d))).astype(np.float32)
    dO = make_grad_output(B, H, L, d, dtype, seed=710)
    g = to_dev(x, dtype)
    r = nats.hybrid_attn_bwd(*(g[k] for k in ("Q", "K", "V", "alpha", "beta", "mask")),
                             torch.from_numpy(dO).to(g["Q"].dtype).cuda(), linear_op=linear_op,
                             initial_state=torch.from_numpy(S0).cuda(), want=("d_initial_state",))
    ref = nbw.hybrid_bwd(x["Q"], x["K"], x["V"], x["alpha"], x["beta"], x["mask"], dO, S0=S0, linear_op=int(linear_op))
    torch.cuda.synchronize()
    for key, want in (("dQ", "dQ"), ("dK", "dK"), ("dV", "dV"), ("dbeta", "dbeta"), ("d_initial_state", "dS0")):
        assert rel_err(host(r[key]), ref[want]) <= 1e-4, key      # the bar of the fp32-accurate gradients
    # dalpha is a sum of fp32 terms of the size of its largest partial sums, divided by alpha: at alpha = 1e-3 that
    # rounding (2^-24 of the terms) counts a thousandfold, so the bar is held before the division
    assert rel_err(host(r["dalpha"]) * x["alpha"], ref["dalpha"] * x["alpha"]) <= 1e-4
