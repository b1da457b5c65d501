"""Workspaces that the calls refuse, and one that they take."""
import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb

pytestmark = pytest.mark.gpu
NAMES = ("state", "k_cache", "v_cache", "cache_len", "q", "k", "v", "alpha", "beta", "mask")


def _step(B, H, d, cap, dtype=torch.bfloat16, seed=0, length=None):
    gen = torch.Generator().manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    unit = lambda *s: torch.nn.functional.normalize(rnd(*s), dim=-1).to(dtype)
    x = dict(state=0.02 * rnd(B, H, d, d), k_cache=unit(B, H, cap, d), v_cache=rnd(B, H, cap, d).to(dtype),
             cache_len=torch.full((B, H), cap - 1 if length is None else length, dtype=torch.int32), q=unit(B, H, d), k=unit(B, H, d),
             v=rnd(B, H, d).to(dtype), alpha=torch.sigmoid(2 + rnd(B, H)), beta=torch.sigmoid(rnd(B, H)),
             mask=torch.zeros(B, H, dtype=torch.uint8))
    return {k: v.cuda() for k, v in x.items()}


@pytest.mark.parametrize("kind", ["cpu", "expanded", "strided"])
def test_a_workspace_that_is_not_plain_gpu_memory_is_refused(kind):
    """A host pointer, or a view whose elements do not cover that many bytes, must not reach the kernels."""
    x = _step(1, 2, 64, 96)
    n = nb.decode_workspace_bytes(1, 2, 64, 96, nb.NATS_BF16)
    ws = {"cpu": lambda: torch.empty(n, dtype=torch.uint8), "strided": lambda: torch.empty(2 * n, dtype=torch.uint8, device="cuda")[::2],
          "expanded": lambda: torch.empty(1, dtype=torch.uint8, device="cuda").expand(n)}[kind]()
    with pytest.raises(ValueError, match="workspace"):
        nats.hybrid_attn_decode(*(x[k] for k in NAMES), workspace=ws)
    L = 64
    q = torch.zeros(1, 1, L, 64, device="cuda")
    g = torch.zeros(1, 1, L, device="cuda")
    m = torch.zeros(1, 1, L, dtype=torch.uint8, device="cuda")
    n = 1 << 22
    ws = {"cpu": lambda: torch.empty(n, dtype=torch.uint8), "strided": lambda: torch.empty(2 * n, dtype=torch.uint8, device="cuda")[::2],
          "expanded": lambda: torch.empty(1, dtype=torch.uint8, device="cuda").expand(n)}[kind]()
    for call in (lambda: nats.hybrid_attn_fwd(q, q, q, g, g, m, workspace=ws),
                 lambda: nats.hybrid_attn_fwd_ex(q, q, q, g, g, m, workspace=ws),
                 lambda: nats.hybrid_attn_bwd(q, q, q, g, g, m, q, workspace=ws)):
        with pytest.raises(ValueError, match="workspace"):
            call()


def test_a_workspace_of_any_shape_serves():
    x = _step(1, 2, 64, 96)
    y = {k: v.clone() for k, v in x.items()}
    n = (nb.decode_workspace_bytes(1, 2, 64, 96, nb.NATS_BF16) + 63) // 64 * 64
    a = nats.hybrid_attn_decode(*(x[k] for k in NAMES), workspace=torch.empty(n, dtype=torch.uint8, device="cuda"))
    b = nats.hybrid_attn_decode(*(y[k] for k in NAMES), workspace=torch.empty(n // 64, 64, dtype=torch.uint8, device="cuda"))
    assert torch.equal(a, b)
