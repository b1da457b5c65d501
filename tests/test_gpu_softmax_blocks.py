"""The bf16 softmax kernel's two block sizes: 128 queries where those fill the chip, 64 otherwise.  What a query gets does not
depend on the block it is in, so a batch and its members in calls of their own, which take the other size, agree bit for
bit (the linear branch's segments held fixed); a length that no block size divides, counts of 0 and of whole tiles."""
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("want", [(), ("O_nla", "lse")])
@pytest.mark.parametrize("combine_mode", [0, 1])
@pytest.mark.parametrize("routing", [nb.NATS_ROUTE_TOKEN, nb.NATS_ROUTE_CHUNK])
@pytest.mark.parametrize("d", [64, 128])
def test_block_sizes_agree(d, routing, combine_mode, want):
    B, H, L = 4, 16, 1088          # 576 blocks of 128 queries; 144 for a member
    g = to_dev(make_fwd_inputs(B, H, L, d, "bf16", 0.15, seed=1200 + d), "bf16")
    g["mask"][:, 0] = 0            # no softmax token at all
    g["mask"][:, 1] = 0
    g["mask"][:, 1, :64] = 1       # one whole tile
    if routing == nb.NATS_ROUTE_CHUNK:
        g["mask"] = g["mask"][:, :, ::64].contiguous()
    names = ("Q", "K", "V", "alpha", "beta", "mask")
    kw = dict(routing=routing, combine_mode=combine_mode, gdn_segments=2, want=want)
    whole = nats.hybrid_attn_fwd_ex(*(g[k] for k in names), 64, **kw)
    for b in range(B):
        part = nats.hybrid_attn_fwd_ex(*(g[k][b:b + 1].contiguous() for k in names), 64, **kw)
        for key in ("O",) + want:
            assert torch.equal(whole[key][b:b + 1], part[key]), (key, b)
