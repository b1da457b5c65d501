"""The two kernels of the backward pass that walk along the sequence take two slices of 16 value columns per block where one slice per
block makes more blocks than there are CUs (bf16 tensors): the same products in the same order, so a pass over many heads is
bit for bit the passes over a few of them."""
import pytest
import torch

import paper_2602_03681_amd as nats
from nats_inputs import make_fwd_inputs, make_grad_output

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


# B x H x G heads of V, d / 16 slices each, on 256 CUs: 257 .. 264, and the last with one; chunks 1 (the walk's shortest), 2, 3
@pytest.mark.parametrize("B,H,G,d,combine_mode,linear_op", [(33, 1, 1, 128, 0, 0), (11, 1, 3, 128, 1, 0), (33, 1, 1, 128, 0, 1),
                                                            (65, 1, 1, 64, 0, 0), (33, 1, 2, 64, 1, 0), (32, 1, 1, 128, 0, 0)])
@pytest.mark.parametrize("L", [64, 128, 192])
def test_many_heads_as_few(L, B, H, G, d, combine_mode, linear_op):
    g = to_dev(make_fwd_inputs(B, H, L, d, "bf16", 0.2, seed=41), "bf16")
    V = to_dev(make_fwd_inputs(B, H * G, L, d, "bf16", 0.2, seed=42), "bf16")["V"]
    dO = torch.from_numpy(make_grad_output(B, H * G, L, d, "bf16", seed=43)).to(torch.bfloat16).cuda()
    S0 = 0.1 * torch.randn(B, H * G, d, d, generator=torch.Generator().manual_seed(44)).cuda()
    kw = dict(group=G, combine_mode=combine_mode, linear_op=linear_op, want=("d_initial_state",))

    def run(b0, b1):
        a = [t[b0:b1].contiguous() for t in (g["Q"], g["K"], V, g["alpha"], g["beta"], g["mask"], dO)]
        return nats.hybrid_attn_bwd(*a, initial_state=S0[b0:b1].contiguous(), **kw)

    whole, few = run(0, B), [run(b, min(b + 8, B)) for b in range(0, B, 8)]
    torch.cuda.synchronize()
    for key, got in whole.items():
        assert torch.isfinite(got).all(), key
        assert torch.equal(got, torch.cat([f[key] for f in few])), key
