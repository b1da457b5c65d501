"""nats_hybrid_attn_bwd_bf16 refuses outputs that share memory with anything else of the call before it launches anything: the fp32
gradients, its scratch, are read after rows of the rounded ones are written.  (Host-side checks on addresses; nothing is read there.)"""
import ctypes

import pytest

from paper_2602_03681_amd import binding as nb

E_SHAPE = -2
B, H, L, d = 1, 2, 128, 64
INPUTS = ("Q", "K", "V", "alpha", "beta", "mask", "dO")
GRADS = ("dQ", "dK", "dV", "dalpha", "dbeta")
ROUNDED = ("dQ_bf16", "dK_bf16", "dV_bf16")
EXTRA = ("initial_state", "d_initial_state", "g_nla", "g_la", "dscore_nla", "dscore_la", "Q_nla", "K_nla", "dQ_nla", "dK_nla", "w_nla",
         "w_la", "dw_nla", "dw_la")


def sizes(G):
    tok, v = B * H * L, B * H * G * L * d
    n = dict.fromkeys(("Q", "K", "dQ_bf16", "dK_bf16"), 2 * tok * d)
    n.update(dict.fromkeys(("dQ", "dK"), 4 * tok * d), **dict.fromkeys(("V", "dO", "dV_bf16", "Q_nla", "K_nla"), 2 * v))
    n.update(dict.fromkeys(("dV", "dQ_nla", "dK_nla"), 4 * v), **dict.fromkeys(("alpha", "beta", "dalpha", "dbeta", "g_nla", "g_la"), 4 * tok))
    n.update(dict.fromkeys(("initial_state", "d_initial_state"), 4 * B * H * G * d * d), mask=tok)
    n.update(dict.fromkeys(("dscore_nla", "dscore_la"), 4 * tok // 64), **dict.fromkeys(("w_nla", "w_la", "dw_nla", "dw_la"), 4 * tok * G))
    return n


def call(G, move):
    """every array 256 MiB apart from the next but those that `move` puts elsewhere"""
    p = nb.make_fwd_params(B, H, L, d, 64, nb.NATS_BF16, combine_mode=1, group=G)
    names = INPUTS + GRADS + EXTRA + ROUNDED + ("workspace",)
    at = {k: (i + 1) << 28 for i, k in enumerate(names)}
    n = nb.load_library().nats_hybrid_attn_bwd_workspace_bytes(ctypes.byref(p))
    assert 0 < n < 1 << 28
    at.update({k: f(at) for k, f in move.items()})
    ex = nb.BwdExtra(*(at[k] for k in EXTRA))
    lib = nb.load_library()
    st = lib.nats_hybrid_attn_bwd_bf16(ctypes.byref(p), *(at[k] for k in INPUTS + GRADS), ctypes.byref(ex), *(at[k] for k in ROUNDED),
                                       at["workspace"], n, None)
    return st, lib.nats_last_error().decode()


SIX = ROUNDED + GRADS[:3]
PAIRS = [(a, b) for i, a in enumerate(SIX) for b in SIX[i + 1:] + INPUTS + GRADS[3:] + EXTRA]


@pytest.mark.parametrize("G", [1, 3])
@pytest.mark.parametrize("a,b", PAIRS)
def test_overlaps_are_refused(a, b, G):
    n = sizes(G)
    # the same place; a's first bytes in b's last ones; b's first in a's last
    for shift in (0, n[b] - 16 - n[b] % 16, 16 - n[a]):
        st, msg = call(G, {a: lambda at: at[b] + shift})
        assert st == E_SHAPE and ("share memory" in msg or "alias" in msg), (a, b, shift, st, msg)


@pytest.mark.parametrize("a", SIX)
def test_overlaps_with_the_workspace_are_refused(a):
    for shift in (0, 4096, 16 - sizes(1)[a]):
        st, msg = call(1, {a: lambda at: at["workspace"] + shift})
        assert st == E_SHAPE and "workspace" in msg, (a, shift, st, msg)


def test_neighbours_are_not():
    """arrays that touch and do not overlap get as far as the next refusal (g_la with routing per chunk), for each of the six"""
    lib = nb.load_library()
    n = sizes(1)
    p = nb.make_fwd_params(B, H, L, d, 64, nb.NATS_BF16, routing=nb.NATS_ROUTE_CHUNK)
    names = ROUNDED + GRADS + INPUTS
    at, end = {}, 1 << 20
    for k in names + ("g_la",):
        at[k] = end
        end += n[k] if k != "mask" else 16
    ws_bytes = lib.nats_hybrid_attn_bwd_workspace_bytes(ctypes.byref(p))
    ex = nb.BwdExtra(None, None, None, at["g_la"])
    st = lib.nats_hybrid_attn_bwd_bf16(ctypes.byref(p), *(at[k] for k in INPUTS + GRADS), ctypes.byref(ex), *(at[k] for k in ROUNDED), end,
                                       ws_bytes, None)
    assert st == -6 and "g_la" in lib.nats_last_error().decode()   # NATS_ERR_UNSUPPORTED
