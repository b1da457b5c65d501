"""The automatic number of segments of the linear branch's chunk recurrence where it is more than one (the rule itself:
test_segment_rule.py): state and rows agree with those of one segment, to the fp16 operands and hand-off of both."""
import pytest
import torch

import paper_2602_03681_amd as nats
from nats_inputs import make_fwd_inputs

from gpu_util import host, rel_err, to_dev
from test_segment_rule import segments

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,L,d", [(2, 1024, 128), (3, 1216, 128), (1, 1280, 64), (85, 1024, 64), (1, 4096, 64), (1, 8192, 128)])
def test_automatic_segments(H, L, d):
    assert segments(H, L, d) > 1
    g = to_dev(make_fwd_inputs(1, H, L, d, "bf16", 0.05, seed=1300 + L), "bf16")
    x = tuple(g[k] for k in ("Q", "K", "V", "alpha", "beta", "mask"))
    auto, one = (nats.hybrid_attn_fwd_ex(*x, 64, gdn_segments=n, want=("final_state", "O_la")) for n in (0, 1))
    torch.cuda.synchronize()
    assert rel_err(host(auto["final_state"]), host(one["final_state"])) <= 4e-3   # operand copies of the state are fp16 (2^-11 of values up to 8 RMS)
    assert rel_err(host(auto["O_la"]), host(one["O_la"])) <= 4e-3
