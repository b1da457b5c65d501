"""The linear branch in one pass (a block per one or two slices of 16 value columns) against the same branch as one segment of the
other kernel, which gdn_segments = 1 asks for: both widths, one and two slices per block, every remainder of the staging
wavefronts' three register sets, head grouping, heads that no multiple of eight is, states in and out, the variants."""
import numpy as np
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs

from gpu_util import TOL, host, launched, oracle_fwd, rel_err, to_dev

pytestmark = pytest.mark.gpu

BOUND = 4e-3   # of the RMS: operand copies of the state, U and the handed-over rows are fp16 (2^-11 of values up to 8 RMS)


@pytest.mark.parametrize("H,G,chunks,d,slices", [
    (1, 1, 1, 128, 1), (2, 1, 2, 128, 1), (3, 1, 3, 128, 1), (9, 1, 4, 128, 1), (5, 2, 5, 128, 1), (18, 1, 19, 128, 1),
    (34, 1, 2, 128, 2), (17, 2, 7, 128, 2),
    (1, 1, 1, 64, 1), (3, 1, 5, 64, 1), (7, 3, 6, 64, 1), (66, 1, 3, 64, 2), (80, 1, 4, 64, 2),
])
@pytest.mark.parametrize("variant", ["plain", "gated", "chunk"])
def test_one_pass_and_one_segment_agree(H, G, chunks, d, slices, variant):
    L = 64 * chunks
    x = make_fwd_inputs(1, H, L, d, "bf16", 0.15, seed=2100 + 10 * H + chunks)
    g = to_dev(x, "bf16")
    rng = np.random.default_rng(d + H)
    V = torch.from_numpy(rng.standard_normal((1, H * G, L, d)).astype(np.float32)).to(torch.bfloat16).cuda()
    S0 = torch.from_numpy((0.3 * rng.standard_normal((1, H * G, d, d))).astype(np.float32)).cuda()
    kw = dict(group=G, want=("final_state", "O_la"), initial_state=S0, la_scale=0.75)
    if variant == "gated":
        kw.update(linear_op=1)
    mask = g["mask"]
    if variant == "chunk":
        mask = mask[:, :, ::64].contiguous()
        kw.update(routing=nb.NATS_ROUTE_CHUNK)
    args = (g["Q"], g["K"], V, g["alpha"], g["beta"], mask, 64)
    assert nb.linear_scan_form(nb.make_fwd_params(1, H, L, d, 64, nb.NATS_BF16, group=G)) == (1, slices)
    auto, kernels = launched(lambda: nats.hybrid_attn_fwd_ex(*args, **kw))
    assert "gdn_slice_scan" in kernels and "gdn_seg_pass1" not in kernels
    one, kernels = launched(lambda: nats.hybrid_attn_fwd_ex(*args, gdn_segments=1, **kw))
    assert "gdn_seg_pass1" in kernels and "gdn_slice_scan" not in kernels
    for key in ("final_state", "O_la"):
        assert rel_err(host(auto[key]), host(one[key])) <= BOUND, key
    # the two heads of a group read the same shared inputs: each as a call of its own
    if G > 1 and variant == "plain":
        kw.update(group=1, initial_state=S0[:, ::G].contiguous())
        own = nats.hybrid_attn_fwd_ex(g["Q"], g["K"], V[:, ::G].contiguous(), *args[3:], **kw)
        assert rel_err(host(auto["O_la"][:, ::G]), host(own["O_la"])) <= BOUND


@pytest.mark.parametrize("H,L,d", [(3, 1216, 128), (40, 256, 128), (4, 448, 64)])
def test_one_pass_against_the_oracle(H, L, d):
    x = make_fwd_inputs(1, H, L, d, "bf16", 0.1, seed=77 + L)
    g = to_dev(x, "bf16")
    r, kernels = launched(lambda: nats.hybrid_attn_fwd_ex(*(g[k] for k in ("Q", "K", "V", "alpha", "beta", "mask")), 64,
                                                          want=("final_state", "O_la")))
    assert "gdn_slice_scan" in kernels
    ref = oracle_fwd(x, want=("O_la", "S"))
    assert rel_err(host(r["O_la"]), ref["O_la"]) <= TOL["bf16"]
    assert rel_err(host(r["final_state"]), ref["S"]) <= TOL["bf16"]
