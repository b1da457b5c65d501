"""The backward pass through Eq. 21's merge on bf16 tensors: the kernels take the bf16 tensors beside fp32 gradients of
the branches' rows.  A bf16 number is exact in fp32 and in the products' terms, so the same values handed over as fp32
tensors give the same gradients up to the order of fp32 sums (1e-5 of a gradient's RMS; the kernels' own distance from
the 64-bit oracle is held to 1e-4 elsewhere)."""
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs, make_grad_output

from gpu_util import host, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("routing", [nb.NATS_ROUTE_TOKEN, nb.NATS_ROUTE_CHUNK])
@pytest.mark.parametrize("combine_mode,group,math", [(1, 1, nb.NATS_MATH_AUTO), (1, 2, nb.NATS_MATH_AUTO),
                                                     (2, 3, nb.NATS_MATH_AUTO), (1, 2, nb.NATS_MATH_FP32)])
@pytest.mark.parametrize("d,L", [(64, 64), (64, 192), (128, 320)])
def test_merge_gradients_of_bf16_tensors(d, L, combine_mode, group, math, routing):
    B, H = 1, 2
    x = make_fwd_inputs(B, H, L, d, "bf16", 0.2, seed=900 + d + L)
    g = to_dev(x, "bf16")
    gen = torch.Generator().manual_seed(L)
    V = torch.randn(B, H * group, L, d, generator=gen).bfloat16().cuda()
    w = torch.rand(2, B, H * group, L, generator=gen).cuda()
    dO = torch.from_numpy(make_grad_output(B, H * group, L, d, "bf16", seed=901)).bfloat16().cuda()
    mask = g["mask"][:, :, ::64].contiguous() if routing == nb.NATS_ROUTE_CHUNK else g["mask"]
    r = [nats.hybrid_attn_bwd(g["Q"].to(t), g["K"].to(t), V.to(t), g["alpha"], g["beta"], mask, dO.to(t), group=group,
                              combine_mode=combine_mode, routing=routing, math=math, w_nla=w[0], w_la=w[1])
         for t in (torch.bfloat16, torch.float32)]
    torch.cuda.synchronize()
    # a weight's gradient is divided by the RMS of its row, which multiplies the rounding of the rows it comes from by 10 to
    # 100 where a first token's row is small (1.1e-5 to 2.9e-5 from the 64-bit oracle with either type): the general bar
    for key, tol in (("dQ", 1e-5), ("dK", 1e-5), ("dV", 1e-5), ("dalpha", 1e-5), ("dbeta", 1e-5), ("dw_nla", 1e-4), ("dw_la", 1e-4)):
        assert rel_err(host(r[0][key]), host(r[1][key])) <= tol, key
