"""The kernel that rounds gradients behind the backward pass is in the per-kernel times where it is launched, and nowhere else."""
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("way,launches", [("fp32_gradients", 0), ("rounded_by_the_last_writers", 0), ("chunk", 1), ("group", 1), ("members", 1)])
def test_rounding_is_listed_where_it_is_launched(way, launches):
    B, H, L, d, G = 1, 2, 128, 64, 2 if way in ("group", "members") else 1
    g = to_dev(make_fwd_inputs(B, H, L, d, "bf16", 0.3, seed=91), "bf16")
    gen = torch.Generator().manual_seed(92)
    V, dO = (torch.randn(B, H * G, L, d, generator=gen).bfloat16().cuda() for _ in range(2))
    kw = dict(group=G, grads_bf16=way != "fp32_gradients")
    mask = g["mask"]
    if way == "chunk":
        mask = mask[:, :, ::64].contiguous()
        kw.update(routing=nb.NATS_ROUTE_CHUNK)
    if way == "members":    # a workspace of one member's pass
        n = nb.load_library().nats_hybrid_attn_bwd_workspace_bytes(nb.make_fwd_params(B, H, L, d, 64, nb.NATS_BF16, group=G))
        kw.update(workspace=torch.empty(n, dtype=torch.uint8, device="cuda"))
    nb.profile_begin(256)
    nats.hybrid_attn_bwd(g["Q"], g["K"], V, g["alpha"], g["beta"], mask, dO, **kw)
    torch.cuda.synchronize()
    kernels = nb.profile_end(32)
    assert kernels.get("round_bf16", {"launches": 0})["launches"] == launches, sorted(kernels)
    assert kernels["gdn_chunk_grads"]["launches"] == (G if way == "members" else 1)
