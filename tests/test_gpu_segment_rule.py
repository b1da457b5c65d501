"""The linear branch in segments where a call chooses them (the rule itself: test_scan_form.py): state and rows agree with those of one
segment, to the fp16 operands and hand-off of both."""
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs

from gpu_util import host, launched, rel_err, to_dev

pytestmark = pytest.mark.gpu

BOUND = 4e-3   # operand copies of the state are fp16 (2^-11 of values up to 8 RMS)


def agree(n, H, L, d, G=1, **kw):
    g = to_dev(make_fwd_inputs(1, H, L, d, "bf16", 0.05, seed=1300 + L), "bf16")
    V = to_dev(make_fwd_inputs(1, H * G, L, d, "bf16", 0.05, seed=1301 + L), "bf16")["V"]
    mask = g["mask"][:, :, ::64].contiguous() if kw.get("routing") else g["mask"]
    x = (g["Q"], g["K"], V, g["alpha"], g["beta"], mask)
    run = lambda n: nats.hybrid_attn_fwd_ex(*x, 64, gdn_segments=n, group=G, want=("final_state", "O_la"), **kw)
    auto, kernels = launched(lambda: run(0))
    assert kernels >= {"gdn_seg_pass1", "gdn_seg_pass2", "gdn_seg_fix"} and "gdn_slice_scan" not in kernels
    assert nb.linear_scan_form(nb.make_fwd_params(1, H, L, d, 64, nb.NATS_BF16, group=G, **kw)) == (n, 0)
    one, kernels = launched(lambda: run(1))
    assert "gdn_seg_pass1" in kernels and "gdn_seg_pass2" not in kernels
    assert rel_err(host(auto["final_state"]), host(one["final_state"])) <= BOUND
    assert rel_err(host(auto["O_la"]), host(one["O_la"])) <= BOUND


@pytest.mark.parametrize("H,L,d,n", [(66, 1152, 128, 3), (48, 4160, 128, 5), (33, 1792, 128, 7), (18, 4288, 128, 10), (1, 8192, 128, 22),
                                     (32, 2432, 64, 8), (24, 3264, 64, 9), (1, 4096, 64, 16)])
def test_automatic_segments(H, L, d, n):
    agree(n, H, L, d)


@pytest.mark.parametrize("L,d,n", [(2560, 128, 10), (2048, 64, 8)])
@pytest.mark.parametrize("variant", ["gated", "chunk", "group", "frozen"])
def test_variants_in_segments(variant, L, d, n):
    agree(n, 2, L, d, **{"gated": dict(linear_op=1), "chunk": dict(routing=nb.NATS_ROUTE_CHUNK), "group": dict(G=2),
                         "frozen": dict(freeze_on_softmax=True)}[variant])
