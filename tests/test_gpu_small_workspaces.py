"""Calls on a workspace smaller than the reported one that they still take: the same results by the way that needs less."""
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs

from gpu_util import TOL, host, oracle_fwd, rel_err, stored, to_dev
from test_workspace_sizes import sizes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_fp32_forward_token_by_token(dtype):
    B, H, L, d = 1, 2, 320, 64
    x = make_fwd_inputs(B, H, L, d, dtype, 0.2, seed=77)
    g = to_dev(x, dtype)
    args = [g[k] for k in ("Q", "K", "V", "alpha", "beta", "mask")]
    n = sizes(B, H, L, d, nb.NATS_F32 if dtype == "f32" else nb.NATS_BF16)
    ws = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    r = nats.hybrid_attn_fwd_ex(*args, 64, math=nb.NATS_MATH_FP32, want=("O_la", "final_state"), workspace=ws[:n])
    assert bool((ws[n:] == 0xA5).all())
    ref = oracle_fwd(x, want=("O_la", "S"))
    assert rel_err(host(r["O"]), ref["O"], stored(dtype)) <= TOL[dtype]
    assert rel_err(host(r["O_la"]), ref["O_la"]) <= 1e-5 and rel_err(host(r["final_state"]), ref["S"]) <= 1e-5
    with pytest.raises(nb.NatsError, match="needed"):
        nats.hybrid_attn_fwd_ex(*args, 64, math=nb.NATS_MATH_FP32, workspace=ws[:n - 1])
