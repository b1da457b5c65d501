"""The calls of the hybrid-attention operator whose speed is watched, as a user's program makes them.

Every case is one pass through the package's public entry points on seeded synthetic inputs of the workloads'
distributions: q, k of unit length per token and head, v ~ N(0,1), alpha = sigmoid(N(2, 0.5^2)), beta = sigmoid(N(0,1)),
a routing mask with a given share of softmax tokens (or chunks).  Kinds of pass:

  fwd           one call of hybrid_attn_fwd, output and workspace kept by the caller (routing per token, plain sum)
  prefill       one call of hybrid_attn_fwd_ex as a server makes it before generation: merge of Eq. 21 with the weights
                of Eq. 22, a state carried in, the final state and the compacted cache handed out
  layer         routing per chunk as the method decides it: route_chunks on the layer's input, then the forward with
                head grouping and the merge of Eq. 21 / 22 under the mask it returns
  train         a training step's share: hybrid_attn (the autograd wrapper) forwards and backwards, gradients of every
                input; with routing per chunk also of the chunk scores
  decode        tokens of generation with routing per token, from cache lengths that are set back at the start
  decode_chunk  one chunk of generation with routing per chunk: 64 tokens and the commit
"""
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb

C = 64


def listed():
    return [
        # the smallest forward: a short prompt in fp32, where launches and the length of the dependent chain count
        dict(name="fwd_tiny_f32", kind="fwd", dtype="f32", B=1, H=2, L=256, d=64, p=0.10, runs=0, linear_op=0),
        # an ordinary batch of short sequences, narrow heads
        dict(name="fwd_short_bf16", kind="fwd", dtype="bf16", B=4, H=8, L=2048, d=64, p=0.10, runs=0, linear_op=0),
        # the benchmark's forward
        dict(name="fwd_headline_bf16", kind="fwd", dtype="bf16", B=2, H=16, L=8192, d=128, p=0.05, runs=0, linear_op=0),
        # long context, few softmax tokens and some that stand together
        dict(name="fwd_long_bf16", kind="fwd", dtype="bf16", B=1, H=16, L=32768, d=128, p=0.02, runs=8, linear_op=0),
        # three prompts of a ragged length continued from a state, before generation starts
        dict(name="prefill_ragged_bf16", kind="prefill", dtype="bf16", B=3, H=6, L=1216, d=128, p=0.20),
        # a whole layer's attention in the paper's geometry: 6 linear heads, 12 softmax heads, hidden width 1024
        dict(name="layer_chunk_bf16", kind="layer", dtype="bf16", B=4, H=6, group=2, L=4096, d=128, d_model=1024, p=0.10),
        # a training step's forward and backward on the benchmark's shapes
        dict(name="train_token_bf16", kind="train", dtype="bf16", B=2, H=16, group=1, L=8192, d=128, p=0.05,
             routing="token", combine_mode=0),
        # a training step in the paper's geometry and context length, merge of Eq. 21 with trained weights and scores
        dict(name="train_chunk_bf16", kind="train", dtype="bf16", B=4, H=6, group=2, L=4096, d=128, p=0.10,
             routing="chunk", combine_mode=1),
        # a small training step in fp32, ragged length, narrow heads
        dict(name="train_small_f32", kind="train", dtype="f32", B=2, H=3, group=1, L=704, d=64, p=0.15,
             routing="token", combine_mode=0),
        # generation for a full batch with caches of very different lengths, the step on a caller's workspace
        dict(name="decode_batch_bf16", kind="decode", dtype="bf16", B=64, H=16, d=128, p=0.05, lo=64, hi=2048, tokens=8,
             workspace=True),
        # generation for one user: the plain call, where latency counts
        dict(name="decode_single_bf16", kind="decode", dtype="bf16", B=1, H=16, d=128, p=0.05, lo=900, hi=1100, tokens=16,
             workspace=False),
        # generation in the paper's geometry with routing per chunk: a whole chunk and its commit
        dict(name="decode_chunk_bf16", kind="decode_chunk", dtype="bf16", B=8, H=12, d=128, p=0.10, lo=64, hi=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _length(rng, lo, hi, head_tokens, heads):
    """A multiple of 64 between lo and hi whose product with `heads` stays within head_tokens."""
    hi = max(lo, min(hi, head_tokens // heads))
    return max(1, _log_int(rng, lo, hi) // C) * C


def draw(rng):
    kind = rng.choice(["fwd", "fwd", "fwd", "prefill", "layer", "train", "train", "decode", "decode", "decode_chunk"])
    d = rng.choice([64, 128])
    p = round(0.02 * (0.4 / 0.02) ** rng.random(), 3)
    if kind == "fwd":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        B, H = rng.randint(1, 5), rng.randint(1, 16)
        L = _length(rng, 64, 32768 if dtype == "bf16" else 4096, 1 << 18 if dtype == "bf16" else 1 << 16, B * H)
        return dict(kind=kind, dtype=dtype, B=B, H=H, L=L, d=d, p=p, runs=rng.choice([0, 0, 3]) if L >= 256 else 0,
                    linear_op=rng.choice([0, 0, 0, 1]))
    if kind == "prefill":
        B, H = rng.randint(1, 6), rng.randint(2, 16)
        return dict(kind=kind, dtype="bf16", B=B, H=H, L=_length(rng, 128, 8192, 1 << 17, B * H), d=d, p=p)
    if kind == "layer":
        B, H, G = rng.randint(1, 5), rng.randint(2, 9), rng.randint(1, 3)
        return dict(kind=kind, dtype="bf16", B=B, H=H, group=G, L=_length(rng, 256, 8192, 1 << 17, B * H * G), d=d,
                    d_model=rng.choice([512, 1024, 1536, 2048]), p=p)
    if kind == "train":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        B, H, G = rng.randint(1, 4), rng.randint(1, 12), rng.randint(1, 3)
        return dict(kind=kind, dtype=dtype, B=B, H=H, group=G,
                    L=_length(rng, 128, 8192, 1 << 17 if dtype == "bf16" else 1 << 15, B * H * G), d=d,
                    p=min(p, 0.2), routing=rng.choice(["token", "chunk"]), combine_mode=rng.choice([0, 1]))
    B = _log_int(rng, 1, 64 if kind == "decode" else 16)
    H = rng.randint(2, 16)
    lo = _log_int(rng, 16, 512)
    case = dict(kind=kind, dtype="bf16", B=B, H=H, d=d, p=p, lo=lo, hi=_log_int(rng, lo, 2048))
    if kind == "decode":
        case.update(tokens=rng.randint(4, 12), workspace=rng.choice([True, False]))
    return case


def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


class _Draws:
    """Numbers of the workloads' distributions, on the GPU."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dtype = dtype

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device="cuda")

    def rows(self, *shape):
        return self.normal(*shape).to(self.dtype)

    def unit_rows(self, *shape):
        return torch.nn.functional.normalize(self.normal(*shape), dim=-1).to(self.dtype)

    def alpha(self, *shape):
        return torch.sigmoid(2.0 + 0.5 * self.normal(*shape))

    def beta(self, *shape):
        return torch.sigmoid(self.normal(*shape))

    def mask(self, p, *shape):
        return (torch.rand(*shape, generator=self.g, device="cuda") < p).to(torch.uint8)

    def ints(self, lo, hi, *shape):
        return torch.randint(lo, hi + 1, shape, generator=self.g, device="cuda", dtype=torch.int32)


def _tokens(r, case, G=1):
    B, H, L, d = (case[k] for k in ("B", "H", "L", "d"))
    return dict(Q=r.unit_rows(B, H, L, d), K=r.unit_rows(B, H, L, d), V=r.rows(B, H * G, L, d), alpha=r.alpha(B, H, L),
                beta=r.beta(B, H, L))


def _token_mask(r, case):
    B, H, L = (case[k] for k in ("B", "H", "L"))
    mask = r.mask(case["p"], B, H, L)
    if case.get("runs"):          # softmax tokens in runs of 16
        at = r.ints(1, L - 16, B, H, case["runs"]).long()[..., None] + torch.arange(16, device="cuda")
        mask.scatter_(2, at.flatten(2), 1)
    mask[:, :, 0] = 1
    return mask


def _fwd_workspace(case, **kw):
    prm = nb.make_fwd_params(case["B"], case["H"], case["L"], case["d"], C,
                             nb.NATS_BF16 if case["dtype"] == "bf16" else nb.NATS_F32, **kw)
    return torch.empty(nb.fwd_workspace_bytes(prm), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    kind, dt = case["kind"], _torch_dtype(case)
    B, H, d = case["B"], case["H"], case["d"]
    r = _Draws(seed, dt)
    s = {"case": case}
    if kind == "fwd":
        s["x"] = _tokens(r, case)
        s["x"]["mask"] = _token_mask(r, case)
        s["workspace"] = _fwd_workspace(case, linear_op=case["linear_op"])
        s["out"] = torch.empty_like(s["x"]["Q"])
    elif kind == "prefill":
        s["x"] = _tokens(r, case)
        s["x"]["mask"] = _token_mask(r, case)
        s["state"] = 0.02 * r.normal(B, H, d, d)
        s["W_out"] = r.normal(H, 2, d)
        s["workspace"] = _fwd_workspace(case, combine_mode=1)
    elif kind == "layer":
        G, dm = case["group"], case["d_model"]
        s["x"] = _tokens(r, case, G)
        # input features with a mean of 0.5, and a score layer that turns it into the share p of softmax chunks: the
        # difference of a head's two scores has a deviation of sqrt(2 / 64) over chunks
        s["X"] = (0.5 + r.normal(B, case["L"], dm)).to(dt)
        W_s = r.normal(H, 2, dm) / dm ** 0.5
        W_s -= W_s.mean(-1, keepdim=True)
        shift = float(torch.special.ndtri(torch.tensor(case["p"], dtype=torch.float64))) * (2.0 / C) ** 0.5
        W_s[:, 0] += shift / (0.5 * dm)
        s["W_s"] = W_s
        s["W_out"] = r.normal(H * G, 2, d)
        s["workspace"] = _fwd_workspace(case, combine_mode=1, routing=nb.NATS_ROUTE_CHUNK, group=G)
    elif kind == "train":
        G, L = case["group"], case["L"]
        s["x"] = _tokens(r, case, G)
        s["dO"] = r.rows(B, H * G, L, d)
        s["opts"] = dict(group=G, combine_mode=case["combine_mode"])
        if case["combine_mode"]:
            w = torch.sigmoid(r.normal(B, H * G, L))
            s["x"].update(w_nla=w, w_la=1.0 - w)
        if case["routing"] == "chunk":
            s["opts"]["routing"] = nb.NATS_ROUTE_CHUNK
            s["mask"] = r.mask(case["p"], B, H, L // C)
            s["mask"][:, :, 0] = 1
            s["x"].update(score_nla=r.normal(B, H, L // C), score_la=r.normal(B, H, L // C))
        else:
            s["mask"] = _token_mask(r, case)
        for t in s["x"].values():
            t.requires_grad_()
    else:
        n = case["tokens"] if kind == "decode" else C
        cap = case["hi"] + n
        lens = r.ints(case["lo"], case["hi"], B, 1).expand(B, H).contiguous()
        s["len0"], s["len"] = lens, lens.clone()
        s["state"] = 0.02 * r.normal(B, H, d, d)
        s["k_cache"], s["v_cache"] = r.unit_rows(B, H, cap, d), r.rows(B, H, cap, d)
        token = dict(q=r.unit_rows(n, B, H, d), k=r.unit_rows(n, B, H, d), v=r.rows(n, B, H, d), alpha=r.alpha(n, B, H),
                     beta=r.beta(n, B, H), out=torch.empty(n, B, H, d, dtype=dt, device="cuda"))
        if kind == "decode":
            token["mask"] = r.mask(case["p"], n, B, H)
            s["workspace"] = None
            if case["workspace"]:
                s["workspace"] = torch.empty(nb.decode_workspace_bytes(B, H, d, cap, nb.NATS_BF16), dtype=torch.uint8,
                                             device="cuda")
        else:
            s["mask_c"] = r.mask(case["p"], B, H)
            s["st"] = dict(state=s["state"], state_start=torch.empty_like(s["state"]),
                           chunk_decay=torch.ones(B, H, device="cuda"),
                           chunk_pos=torch.zeros(B, H, dtype=torch.int32, device="cuda"), k_cache=s["k_cache"],
                           v_cache=s["v_cache"], cache_len=s["len"])
        s["tokens"] = [{k: v[t] for k, v in token.items()} for t in range(n)]
        s["o"] = token["out"]
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "fwd":
        x = s["x"]
        return nats.hybrid_attn_fwd(x["Q"], x["K"], x["V"], x["alpha"], x["beta"], x["mask"], C,
                                    linear_op=case["linear_op"], out=s["out"], workspace=s["workspace"])
    if kind == "prefill":
        return nats.hybrid_attn_fwd_ex(*(s["x"][k] for k in ("Q", "K", "V", "alpha", "beta", "mask")), C, combine_mode=1,
                                       W_out=s["W_out"], initial_state=s["state"],
                                       want=("final_state", "Kc", "Vc", "n_s"), workspace=s["workspace"])
    if kind == "layer":
        mask, scores = nats.route_chunks(s["X"], s["W_s"], C)
        r = nats.hybrid_attn_fwd_ex(*(s["x"][k] for k in ("Q", "K", "V", "alpha", "beta")), mask, C,
                                    routing=nb.NATS_ROUTE_CHUNK, combine_mode=1, W_out=s["W_out"], group=case["group"],
                                    workspace=s["workspace"])
        return dict(O=r["O"], mask=mask, scores=scores)
    if kind == "train":
        x = s["x"]
        for t in x.values():
            t.grad = None
        O = nats.hybrid_attn(*(x[k] for k in ("Q", "K", "V", "alpha", "beta")), s["mask"], C, **s["opts"],
                             **{k: x[k] for k in ("w_nla", "w_la", "score_nla", "score_la") if k in x})
        O.backward(s["dO"])
        return dict(O=O.detach(), **{"d" + k: t.grad for k, t in x.items()})
    # generation: the caches keep the rows of the prompt, the lengths go back to the prompt's end
    s["len"].copy_(s["len0"])
    if kind == "decode":
        for t in s["tokens"]:
            nats.hybrid_attn_decode(s["state"], s["k_cache"], s["v_cache"], s["len"], t["q"], t["k"], t["v"], t["alpha"],
                                    t["beta"], t["mask"], out=t["out"], workspace=s["workspace"])
    else:
        for t in s["tokens"]:
            nats.hybrid_attn_decode_chunk(s["st"], t["q"], t["k"], t["v"], t["alpha"], t["beta"], out=t["out"])
        nats.hybrid_attn_decode_commit(s["st"], s["mask_c"])
    return dict(o=s["o"], state=s["state"], cache_len=s["len"], k_cache=s["k_cache"], v_cache=s["v_cache"])


def work(case):
    kind = case["kind"]
    B, H, d = case["B"], case["H"], case["d"]
    es = 2 if case["dtype"] == "bf16" else 4
    if kind in ("decode", "decode_chunk"):
        n = case["tokens"] if kind == "decode" else C
        grow = case["p"] * n / 2 if kind == "decode" else n / 2       # rows that came in before a token, on average
        rows = (case["lo"] + case["hi"]) / 2 + grow
        per_token = 8 * d * d + 2 * d * es * rows + 4 * d * es
        return {"bytes": B * H * n * per_token, "flops": B * H * n * (8.0 * d * d + 4.0 * d * rows)}
    L, G, p = case["L"], case.get("group", 1), case["p"]
    n, nG = B * H * L, B * H * G * L
    chunked = kind == "layer" or case.get("routing") == "chunk"
    pairs = nG * (p * L / 2 + (C / 2 if chunked else 0))
    flops = nG * (6.0 * d * d + 6.0 * C * d) + n * (4.0 * C * d + C * C / 3.0) + 4.0 * d * pairs
    nbytes = es * d * (2 * n + 2 * nG) + 8 * n + (n / C if chunked else n)
    if kind == "prefill":
        nbytes += 8 * B * H * d * d + 2 * es * d * n      # states in and out, cache rows (capacity L, cleared) out
    if kind == "layer":
        nbytes += es * B * L * case["d_model"]
        flops += 2.0 * B * L * case["d_model"]
    if kind == "train":     # dO in; the gradients out; each product of the forward has two in the backward
        nbytes += es * d * (2 * n + 2 * nG) + 8 * n + (16 * nG if case["combine_mode"] else 0)
        flops *= 3.0
    return {"bytes": float(nbytes), "flops": flops}


def tolerance(case):
    # Measured: fp32 cases against the fp64 oracle (worst 5e-7 of the 2-norm, dalpha), decode against the step's other
    # form, whose sums run in another order (3e-5, single bf16 roundings that fall the other way: up to one unit in the
    # last place, 2^-7 of a value), bf16 forwards against the fp32 arithmetic path (1.2e-3 from fp16 intermediates and
    # the bf16 rounding of O, 2^-7 of a value at most).
    if case["dtype"] == "f32":
        return {"rel": 4e-6}
    if case["kind"] in ("decode", "decode_chunk"):
        return {"rel": 2e-4, "max": 1.6e-2}
    return {"rel": 5e-3, "max": 2e-2}
