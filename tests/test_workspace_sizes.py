"""Workspace sizes, on the host: what is reported, what is taken.  No call here gets as far as a launch."""
import ctypes
import re

import pytest

from paper_2602_03681_amd import binding as nb

FAKE = ctypes.c_void_p(0x1000)   # checked for alignment only


@pytest.fixture(scope="module")
def lib():
    return nb.load_library()


def needed(call):
    """the size that a call on 16 bytes asks for"""
    assert call(16) == -5                                  # NATS_ERR_WORKSPACE
    return int(re.search(rb"(\d+) needed", nb.load_library().nats_last_error()).group(1))


def sizes(B, H, L, d, dtype):
    """cnt, idx, n_s, Kc, Vc, O_la and the weights, each rounded up to 256 bytes"""
    es, up = (4 if dtype == nb.NATS_F32 else 2), lambda n: (n + 255) // 256 * 256
    n = B * H * L
    return 2 * up(4 * n) + up(4 * B * H) + 2 * up(n * d * es) + up(4 * n * d) + up(8 * n)


@pytest.mark.parametrize("dtype,math", [(nb.NATS_F32, nb.NATS_MATH_AUTO), (nb.NATS_BF16, nb.NATS_MATH_FP32)])
@pytest.mark.parametrize("B,H,L,d", [(1, 2, 64, 64), (2, 8, 4096, 128), (1, 3, 704, 64)])
def test_fp32_forward_takes_a_workspace_without_states(lib, B, H, L, d, dtype, math):
    p = nb.make_fwd_params(B, H, L, d, 64, dtype, math=math)
    reported = nb.fwd_workspace_bytes(p)
    small = needed(lambda n: lib.nats_hybrid_attn_fwd(ctypes.byref(p), *([FAKE] * 7), FAKE, n, None))
    assert small == sizes(B, H, L, d, dtype) < reported


@pytest.mark.parametrize("dtype", [nb.NATS_F32, nb.NATS_BF16])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("B,H,L,d", [(1, 2, 64, 64), (2, 4, 4096, 128)])
def test_grouped_backward_reports_one_size(lib, B, H, L, d, mode, dtype):
    """Member by member, which is what is reported, the size is the same for every group, and that size is taken."""
    size = {}
    for G in (1, 2, 3, 8):
        p = nb.make_fwd_params(B, H, L, d, 64, dtype, group=G, combine_mode=mode)
        size[G] = lib.nats_hybrid_attn_bwd_workspace_bytes(ctypes.byref(p))
        assert needed(lambda n: lib.nats_hybrid_attn_bwd(ctypes.byref(p), *([FAKE] * 12), None, FAKE, n, None)) == size[G]
    assert size[1] < size[2] == size[3] == size[8] < 2 * size[1]
