"""Gradients of bf16 tensors rounded in the kernels that write them last: bit for bit the fp32 gradients of the same pass, rounded, on
every way through the pass (written there, summed over a group there, or rounded behind it)."""
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs, make_grad_output

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("combine_mode", [0, 1])
@pytest.mark.parametrize("case", ["token", "chunk", "token_group", "chunk_group", "members", "own_qk", "by_tokens", "no_softmax", "all_softmax"])
def test_rounded_gradients_are_the_gradients_rounded(case, combine_mode, d):
    H, L = 3, 320
    G = 2 if case in ("token_group", "chunk_group", "members") else 1
    g = to_dev(make_fwd_inputs(1, H, L, d, "bf16", 0.2, seed=31), "bf16")
    big = to_dev(make_fwd_inputs(1, H * G, L, d, "bf16", 0.2, seed=32), "bf16")
    dO = torch.from_numpy(make_grad_output(1, H * G, L, d, "bf16", seed=33)).to(torch.bfloat16).cuda()
    mask = g["mask"]
    if case == "no_softmax": mask = torch.zeros_like(mask)
    if case == "all_softmax": mask = torch.ones_like(mask)
    kw = dict(group=G, combine_mode=combine_mode)
    if case.startswith("chunk"):
        mask = mask[:, :, ::64].contiguous()
        kw.update(routing=nb.NATS_ROUTE_CHUNK)
    if case == "own_qk": kw.update(Q_nla=big["Q"], K_nla=big["K"])
    if case == "by_tokens": kw.update(math=nb.NATS_MATH_FP32)
    if case == "members":    # a workspace of one member's pass: member by member
        prm = nb.make_fwd_params(1, H, L, d, 64, nb.NATS_BF16, combine_mode=combine_mode, group=G)
        n = nb.load_library().nats_hybrid_attn_bwd_workspace_bytes(prm)
        kw.update(workspace=torch.empty(n, dtype=torch.uint8, device="cuda"))
    args = (g["Q"], g["K"], big["V"], g["alpha"], g["beta"], mask, dO, 64)
    want = {k: v.clone() for k, v in nats.hybrid_attn_bwd(*args, **kw).items()}
    got = nats.hybrid_attn_bwd(*args, grads_bf16=True, **kw)
    torch.cuda.synchronize()
    for key, w in want.items():
        if key in ("dQ", "dK", "dV"):
            assert got[key].dtype == torch.bfloat16 and torch.equal(got[key], w.to(torch.bfloat16)), key
        else:
            assert torch.equal(got[key], w), key


def test_fp32_tensors_are_refused():
    g = to_dev(make_fwd_inputs(1, 1, 64, 64, "f32", 0.2, seed=31), "f32")
    with pytest.raises(nb.NatsError):
        nats.hybrid_attn_bwd(*(g[k] for k in ("Q", "K", "V", "alpha", "beta", "mask")), torch.ones_like(g["V"]), grads_bf16=True)
