"""Kc and Vc of hybrid_attn_fwd_ex: the compacted rows first, zeros from there to cap, whatever the memory held; and the C call that
leaves the rows behind the compacted ones as they are."""
import ctypes

import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb
from nats_inputs import make_fwd_inputs

from gpu_util import launched, to_dev

pytestmark = pytest.mark.gpu

# how the mask scan is launched: beside the operands of the bf16 path, beside those of the fp32 path by chunks, by itself
WAYS = {"bf16": ("bf16", {}), "f32": ("f32", {}), "bf16_as_fp32": ("bf16", dict(math=nb.NATS_MATH_FP32)),
        "chunks": ("bf16", dict(routing=nb.NATS_ROUTE_CHUNK)), "group": ("bf16", dict(group=2))}


@pytest.mark.parametrize("way", WAYS)
@pytest.mark.parametrize("mask_kind", ["some", "none", "all"])
@pytest.mark.parametrize("L,cap", [(64, 64), (256, 100), (320, 320), (1216, 1216), (1088, 1500), (320, 1), (1344, 1343),
                                   (64, 5000), (1088, 8300)])
def test_rows_behind_the_compacted_ones_are_zeros(L, cap, mask_kind, way):
    dtype, kw = WAYS[way]
    d, G = (64, 1) if way == "f32" else (128, kw.get("group", 1))
    x = to_dev(make_fwd_inputs(2, 2, L, d, dtype, 0.2, seed=51), dtype)
    V = to_dev(make_fwd_inputs(2, 2 * G, L, d, dtype, 0.2, seed=52), dtype)["V"]
    mask = {"some": x["mask"], "none": torch.zeros_like(x["mask"]), "all": torch.ones_like(x["mask"])}[mask_kind]
    tokens = mask
    if way == "chunks":
        mask = mask[:, :, ::64].contiguous()
        tokens = mask.repeat_interleave(64, dim=2)
    junk = [torch.full((2, 2 * G, cap, d), 7.0, dtype=V.dtype, device="cuda") for _ in range(4)]   # what the new tensors may get
    del junk
    r = nats.hybrid_attn_fwd_ex(x["Q"], x["K"], V, x["alpha"], x["beta"], mask, want=("Kc", "Vc", "n_s"), cap=cap, **kw)
    for b in range(2):
        for h in range(2 * G):
            at = tokens[b, h // G].nonzero().flatten()
            assert int(r["n_s"][b, h // G]) == len(at)
            for got, src in ((r["Kc"][b, h], x["K"][b, h // G]), (r["Vc"][b, h], V[b, h])):
                want = torch.zeros_like(got)
                want[:min(len(at), cap)] = src[at][:cap]
                assert torch.equal(got, want)


@pytest.mark.parametrize("dtype,d,L,apart", [   # apart: the first capacity with it
    # a block per 1024 tokens clears what lies behind L as long as its share is below 1 MB of Kc and Vc together ...
    ("bf16", 128, 64, 64 + 2048), ("bf16", 64, 1024, 1024 + 4096), ("f32", 128, 128, 128 + 1024), ("f32", 64, 1088, 1088 + 4096),
])
def test_large_caches_are_cleared_by_a_launch_of_their_own(dtype, d, L, apart):
    """... which some shares of a few blocks take several times as long over as a launch on all CUs"""
    x = to_dev(make_fwd_inputs(1, 1, L, d, dtype, 0.2, seed=54), dtype)
    args = [x[k] for k in ("Q", "K", "V", "alpha", "beta", "mask")]
    for cap, own in ((L, False), (apart - 1, False), (apart, True), (2 * apart, True)):
        r, kernels = launched(lambda: nats.hybrid_attn_fwd_ex(*args, want=("Kc", "Vc", "n_s"), cap=cap))
        assert ("clear_cache" in kernels) == own, cap
        n = int(r["n_s"][0, 0])
        assert not r["Kc"][0, 0, n:].any() and not r["Vc"][0, 0, n:].any()
        assert torch.equal(r["Vc"][0, 0, :n], x["V"][0, 0][x["mask"][0, 0].bool()])


def test_the_plain_call_leaves_them():
    L, cap, d = 320, 320, 128
    x = to_dev(make_fwd_inputs(1, 2, L, d, "bf16", 0.2, seed=53), "bf16")
    lib = nb.load_library()
    prm = nb.make_fwd_params(1, 2, L, d, 64, nb.NATS_BF16)
    ws = torch.empty(lib.nats_hybrid_attn_fwd_workspace_bytes(ctypes.byref(prm)), dtype=torch.uint8, device="cuda")
    O, kc = torch.empty_like(x["V"]), torch.full((1, 2, cap, d), 7.0, dtype=torch.bfloat16, device="cuda")
    vc = kc.clone()
    extra = nb.FwdExtra()
    extra.Kc, extra.Vc, extra.cap = kc.data_ptr(), vc.data_ptr(), cap
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    st = lib.nats_hybrid_attn_fwd_ex(ctypes.byref(prm), *(p(x[k]) for k in ("Q", "K", "V", "alpha", "beta", "mask")), p(O),
                                     ctypes.byref(extra), p(ws), ws.numel(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    torch.cuda.synchronize()
    for h in range(2):
        n = int(x["mask"][0, h].sum())
        for t, src in ((kc, x["K"]), (vc, x["V"])):
            assert torch.equal(t[0, h, :n], src[0, h][x["mask"][0, h].bool()]) and bool((t[0, h, n:] == 7.0).all())
