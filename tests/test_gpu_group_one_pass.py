"""Head grouping in the backward pass: all output heads in one pass against one call per member of the groups without
grouping (its V, dO, state and weights gathered), whose gradients of the shared inputs are added up here.  The same
kernels on the same numbers: the sums over the members are all that may round differently (1e-6 of a gradient's RMS)."""
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs

from gpu_util import host, rel_err, to_dev

pytestmark = pytest.mark.gpu
SHARED = ("dQ", "dK", "dalpha", "dbeta", "g_nla", "dscore_nla", "dscore_la")


@pytest.mark.parametrize("routing", [nb.NATS_ROUTE_TOKEN, nb.NATS_ROUTE_CHUNK])
@pytest.mark.parametrize("own_qk", [False, True])
@pytest.mark.parametrize("dtype,d,L,G,combine_mode", [("bf16", 128, 192, 2, 1), ("bf16", 64, 320, 3, 0), ("f32", 64, 64, 8, 1),
                                                      ("f32", 128, 128, 2, 0)])
def test_one_pass_is_the_sum_of_its_members(dtype, d, L, G, combine_mode, own_qk, routing):
    B, H = 2, 2
    g = to_dev(make_fwd_inputs(B, H, L, d, dtype, 0.3, seed=950 + d + L), dtype)
    dt = g["Q"].dtype
    gen = torch.Generator().manual_seed(L + G)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    per_head = dict(V=rnd(B, H * G, L, d).to(dt).cuda(), dO=rnd(B, H * G, L, d).to(dt).cuda(),
                    initial_state=(0.1 * rnd(B, H * G, d, d)).cuda())
    if combine_mode:
        per_head.update(w_nla=torch.rand(B, H * G, L, generator=gen).cuda(), w_la=torch.rand(B, H * G, L, generator=gen).cuda())
    if own_qk:
        unit = lambda: torch.nn.functional.normalize(rnd(B, H * G, L, d), dim=-1).to(dt).cuda()
        per_head.update(Q_nla=unit(), K_nla=unit())
    mask = g["mask"][:, :, ::64].contiguous() if routing == nb.NATS_ROUTE_CHUNK else g["mask"]

    def call(t, group):
        t = dict(t)
        V, dO = t.pop("V"), t.pop("dO")
        return nats.hybrid_attn_bwd(g["Q"], g["K"], V, g["alpha"], g["beta"], mask, dO, group=group, routing=routing,
                                    combine_mode=combine_mode, want=("d_initial_state", "g_nla", "dscore_nla", "dscore_la"), **t)

    one = call(per_head, G)
    members = [call({k: v[:, m::G].contiguous() for k, v in per_head.items()}, 1) for m in range(G)]
    torch.cuda.synchronize()
    for key, got in one.items():
        want = sum(m[key] for m in members) if key in SHARED else torch.stack([m[key] for m in members], 2).flatten(1, 2)
        if key == "dscore_nla":   # sums of 64 entries of g_nla that may cancel (over a single chunk they sum to zero)
            bound = 64 * G * 2.0 ** -23 * max(float(m["g_nla"].abs().max()) for m in members)
            assert float((got - want).abs().max()) <= bound
        else:
            assert rel_err(host(got), host(want)) <= 1e-6, key
