"""What this library's speed is measured on: rank steps and single steps as a tensor- or data-parallel program calls
them, through the public binding, from a handful of decoded tokens to the 70B-shape layers and the 1e9-element bucket.

A case is a dict of plain numbers and texts.  ``kind`` names the path:

  steps      p calls of commfuse_rs_step / commfuse_ag_step, one per hop, as a program does that moves the slices itself
             (``noalloc``: commfuse_rs_step_noalloc, the call for serving loops without a workspace)
  rs, ag     one GEMM + reduce-scatter / all-gather + GEMM rank step as one schedule call (one launch, which also carries
             the deliveries), ``rs_pair`` the reduce-scatter under the pairwise schedule
  mlp        the layer pair, forward: all-gather up-projection, then reduce-scatter down-projection of its bf16 result
  backward   the pair's backward pass: two data gradients and two weight gradients
  attn       query-split attention + output projection + reduce-scatter as one schedule call, ``attn_steps`` step by step
  dp         the fp32 gradient-bucket reduce on the ring, ``dp_pair`` under the pairwise schedule

Every buffer the call writes is an output here: the rank's result, every partial sum it sends on, every landed delivery.
"""
from __future__ import annotations

import math

import torch

from paper_2604_24013_amd import binding as cf

DEV = "cuda:0"
ONE_LAUNCH = cf.CF_PERSISTENT | cf.CF_SERIAL | cf.CF_FUSED_COPY
LAYOUTS = {"kn": cf.CF_W_KN, "nk": cf.CF_W_NK}
HEAD_DIM = 128
WORKSPACE_BYTES = (1 << 30) + (1 << 16)     # k-split partials of the largest layer here (8 x 8192 x 3584 fp32) and counters


def listed():
    return [
        # the smallest layer of the benchmark: fp32, two ranks; two launches of a few microseconds
        dict(name="steps_f32_p2", kind="steps", op="rs", dtype="f32", p=2, m_chunk=128, n=256, k=512, layout="kn"),
        # decoding 64 sequences on 8 ranks, 7B down-projection: eight tokens per slice, called hop by hop from a serving loop
        dict(name="decode_rs_7b", kind="steps", op="rs", dtype="bf16", p=8, m_chunk=8, n=4096, k=1376, layout="kn", noalloc=True),
        # the same tokens through the 7B QKV projection as one schedule call
        dict(name="decode_ag_7b", kind="ag", p=8, m_chunk=8, n=1536, k=4096, layout="kn", out="bf16"),
        # 7B prefill, 4096 tokens: down-projection and QKV projection
        dict(name="rs_7b", kind="rs", p=8, m_chunk=512, n=4096, k=1376, layout="kn"),
        dict(name="ag_7b", kind="ag", p=8, m_chunk=512, n=1536, k=4096, layout="kn", out="f32"),
        # odd everything: six ranks, pairwise schedule, ragged rows, columns and contraction, weights kept [n x k]
        dict(name="pair_ragged_p6", kind="rs_pair", p=6, m_chunk=390, n=2088, k=1096, layout="nk"),
        # 70B MLP pair, 8192 tokens: forward (the headline workload) and backward
        dict(name="mlp_70b", kind="mlp", p=8, m_chunk=1024, d=8192, f=3584),
        dict(name="backward_70b", kind="backward", p=8, m_chunk=1024, d=8192, f=3584),
        # 70B attention layer, 8192 positions, 8 of 64 heads per rank
        dict(name="attn_70b", kind="attn", p=8, batch=1, heads=8, seq=8192, n=8192),
        # a small batch of odd-length sequences, four ranks, step by step
        dict(name="attn_steps_ragged", kind="attn_steps", p=4, batch=2, heads=3, seq=1120, n=3072),
        # gradient buckets: 1e9 values, and slices of a million and three (no slice but the first starts on a 16-byte line)
        dict(name="dp_1e9", kind="dp", p=8, chunk=125_000_000),
        dict(name="dp_odd", kind="dp", p=8, chunk=1_000_003),
    ]


def _log_int(rng, lo, hi, mult=1):
    """A multiple of ``mult`` in [lo, hi], spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / mult)) * mult))


def _draw_any(rng):
    kind = rng.choice(["steps", "steps", "rs", "rs", "ag", "ag", "rs_pair", "mlp", "backward", "attn", "attn_steps", "dp", "dp", "dp_pair"])
    c = dict(kind=kind, p=rng.choice([2, 4, 8]))
    if kind == "steps":
        c["op"] = rng.choice(["rs", "ag"])
        c["dtype"] = rng.choice(["bf16", "bf16", "f32"])
    if kind in ("dp", "dp_pair"):
        c["chunk"] = _log_int(rng, 10_000, 125_000_000)
    elif kind in ("attn", "attn_steps"):
        c.update(batch=rng.choice([1, 1, 2, 4]), heads=rng.choice([1, 2, 3, 4, 8]), seq=c["p"] * _log_int(rng, 32, 8192 // c["p"]),
                 n=_log_int(rng, 256, 8192, 8))
    elif kind in ("mlp", "backward"):
        c.update(m_chunk=_log_int(rng, 16, 1024), d=_log_int(rng, 512, 8192, 8), f=_log_int(rng, 256, 3584, 8))
    else:
        if kind == "rs_pair":
            c["p"] = rng.choice([2, 4, 6, 8])
        f32 = c.get("dtype") == "f32"
        c.update(m_chunk=_log_int(rng, 1, 512 if f32 else 1024), n=_log_int(rng, 128, 4096 if f32 else 8192, 8),
                 k=_log_int(rng, 128, 4096 if f32 else 8192, 8), layout=rng.choice(["kn", "nk"]))
        if kind == "ag":
            c["out"] = rng.choice(["bf16", "f32"])
        if kind == "steps" and c["op"] == "rs" and not f32 and c["m_chunk"] * c["n"] <= 1 << 21:
            c["noalloc"] = rng.choice([True, False])
        if kind in ("rs", "ag") and c["m_chunk"] % 2 == 0 and rng.random() < 0.3:
            c["m"] = 2                       # two sub-steps per hop
    return c


def _roughly_us(c):
    w = work(c)
    return (w["flops"] / (1e8 if c.get("dtype") == "f32" else 1e9) + w["bytes"] / 5e6)


def draw(rng):
    limit = max(_roughly_us(c) for c in listed())
    while True:
        c = _draw_any(rng)
        if _roughly_us(c) <= limit:
            return c


# ---------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------------
def work(case):
    c, kind, p = case, case["kind"], case["p"]
    if kind in ("dp", "dp_pair"):
        adds = (p - 1) * c["chunk"]
        touched = adds if kind == "dp" else c["chunk"]           # the bucket's slices that change: read and written
        return {"bytes": 8 * touched + 8 * adds, "flops": adds}  # arrivals: read, and landed
    if kind in ("attn", "attn_steps"):
        rows, hd = c["batch"] * c["seq"], c["heads"] * HEAD_DIM
        part = rows // p * c["n"] * 4
        moved = 3 * rows * hd * 2 + hd * c["n"] * 2 + (p - 1) * part * (2 if kind == "attn" else 1) + p * part
        return {"bytes": moved, "flops": 4 * c["heads"] * rows * c["seq"] * HEAD_DIM + 2 * rows * hd * c["n"]}
    mc = c["m_chunk"]
    if kind == "mlp":
        d, f = c["d"], c["f"]
        up = p * mc * d * 2 + (p - 1) * mc * d * 2 + d * f * 2 + p * mc * f * 2
        down = p * mc * f * 2 + f * d * 2 + (p - 1) * mc * d * 8 + p * mc * d * 4
        return {"bytes": up + down, "flops": 4 * p * mc * d * f}
    if kind == "backward":
        d, f = c["d"], c["f"]
        slices = p * mc * d * 2 + (p - 1) * mc * d * 2           # a gathered operand: read, and its deliveries landed
        dgrad_up = p * mc * f * 2 + d * f * 2 + (p - 1) * mc * d * 8 + p * mc * d * 4
        dgrad_down = slices + d * f * 2 + p * mc * f * 4
        wgrads = 2 * (slices + p * mc * f * 2 + d * f * 4)
        return {"bytes": dgrad_up + dgrad_down + wgrads, "flops": 8 * p * mc * d * f}
    n, k = c["n"], c["k"]
    e = 4 if c.get("dtype") == "f32" else 2
    moved = p * mc * k * e + k * n * e
    if kind == "ag" or c.get("op") == "ag":
        moved += p * mc * n * (2 if c.get("out") == "bf16" else 4) + ((p - 1) * mc * k * e if kind == "ag" else 0)
    else:
        moved += p * mc * n * 4 + (p - 1) * mc * n * 4 * (1 if kind == "steps" else 2)
    return {"bytes": moved, "flops": 2 * p * mc * n * k}


# ---------------------------------------------------------------------------------------------------------------------
# inputs and buffers
# ---------------------------------------------------------------------------------------------------------------------
_workspace = None


def _register_workspace():
    """The workspace a program registers once for all its layers."""
    global _workspace
    if _workspace is None:
        _workspace = torch.empty(WORKSPACE_BYTES, dtype=torch.uint8, device=DEV)
        cf.set_workspace(_workspace, WORKSPACE_BYTES)
        torch.cuda.synchronize()


class _Maker:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, shape, sigma=1.0, dtype="bf16"):
        t = torch.empty(shape, dtype=torch.float32, device=DEV).normal_(0.0, sigma, generator=self.g)
        return t.to(torch.bfloat16) if dtype == "bf16" else t

    def weight(self, k, n, sigma, layout="kn", dtype="bf16"):
        return self.normal((k, n) if layout == "kn" else (n, k), sigma, dtype)


def _out(*shape, dtype=torch.float32):
    return torch.zeros(shape, dtype=dtype, device=DEV)


def _rs_layer(mk, p, mc, n, k, A, W, sigma, layout, rank, kind=cf.CF_KIND_RS, m=1):
    """A reduce-scatter rank step's plan: partial sums arrive with the spread that i products of length k have."""
    stage = [mk.normal((mc, n), sigma * math.sqrt(k * i), "f32") for i in range(1, p)]
    O = _out(mc, n)
    each = [_out(mc, n) for _ in range(p - 1)]
    sends = [_out(mc, n) for _ in range(p - 1)]
    bufs = cf.make_buffers(A, W, O, stage, (None, None), (None, None), None, each, sends)
    desc = cf.layer_desc(p, rank, mc, n, k, "bf16", "f32", LAYOUTS[layout], m=m)
    return dict(desc=desc, kind=kind, bufs=bufs, keep=(A, W, stage), out=dict(O=O, sent=sends, landed=each))


def _ag_layer(mk, p, mc, n, k, own, stage, each, W, layout, out_dtype, rank, m=1):
    O = _out(p * mc, n, dtype=torch.bfloat16 if out_dtype == "bf16" else torch.float32)
    bufs = cf.make_buffers(own, W, O, stage, (None, None), (None, None), None, each)
    desc = cf.layer_desc(p, rank, mc, n, k, "bf16", out_dtype, LAYOUTS[layout], m=m)
    return dict(desc=desc, kind=cf.CF_KIND_AG, bufs=bufs, keep=(own, W, stage), out=dict(O=O, landed=each))


def _gathered(p, mc, width, rank, own):
    """The buffer an all-gather fills: the own slice in row block ``rank``, hop i lands in row block (rank - i) mod p."""
    g = _out(p * mc, width, dtype=torch.bfloat16)
    blk = [g[c * mc:(c + 1) * mc] for c in range(p)]
    blk[rank].copy_(own)
    return g, blk[rank], [blk[(rank - i) % p] for i in range(1, p)]


def _wgrad_layer(p, mc, k, n, own, stage, land, local, left_moves, rank):
    dW = _out(k, n)
    bufs = cf.make_buffers(own, local, dW, stage, (None, None), (None, None), None, land)
    desc = cf.layer_desc(p, rank, mc, n, k, "bf16", "f32")
    return dict(desc=desc, kind=cf.CF_KIND_WGRAD_X if left_moves else cf.CF_KIND_WGRAD_G, bufs=bufs, keep=(own, local, stage, land),
                out=dict(dW=dW))


def _prepare_steps(c, mk, rank):
    p, mc, n, k, dtype = c["p"], c["m_chunk"], c["n"], c["k"], c["dtype"]
    sa, sw = (1.0, 1.0) if dtype == "f32" else (1.0, 0.02)
    W = mk.weight(k, n, sw, c["layout"], dtype)
    desc = cf.layer_desc(p, rank, mc, n, k, dtype, "f32", LAYOUTS[c["layout"]])
    st = dict(desc=desc, W=W)
    if c["op"] == "rs":
        st["A"] = mk.normal((p * mc, k), sa, dtype)
        st["recv"] = [None] + [mk.normal((mc, n), sa * sw * math.sqrt(k * i), "f32") for i in range(1, p)]
        st["out"] = [_out(mc, n) for _ in range(p)]
        st["call"] = cf.rs_step_noalloc if c.get("noalloc") else cf.rs_step
    else:
        st["slices"] = [mk.normal((mc, k), sa, dtype) for _ in range(p)]
        st["out"] = _out(p * mc, n)
    return st


def _prepare_backward(c, mk, rank):
    p, mc, d, f = c["p"], c["m_chunk"], c["d"], c["f"]
    W_up, W_dn = mk.weight(d, f, 0.02), mk.weight(f, d, 0.02)
    G_up, A_dn = mk.normal((p * mc, f)), mk.normal((p * mc, f))          # local operands of the two layers
    G_slices = [mk.normal((mc, d)) for _ in range(p)]                    # output gradient, gathered for the down layer
    X_slices = [mk.normal((mc, d)) for _ in range(p)]                    # activations, gathered for the up layer
    G_all, G_own, G_land = _gathered(p, mc, d, rank, G_slices[0])
    X_all, X_own, X_land = _gathered(p, mc, d, rank, X_slices[0])
    layers = [
        _ag_layer(mk, p, mc, f, d, G_own, G_slices[1:], G_land, W_dn, "nk", "f32", rank),            # dA = AG(G) W_dn^T
        _wgrad_layer(p, mc, f, d, G_own, G_slices[1:], G_land, A_dn, False, rank),                   # dW_dn = A^T AG(G)
        _rs_layer(mk, p, mc, d, f, G_up, W_up, 0.02, "nk", rank),                                    # dX = RS(G_up W_up^T)
        _wgrad_layer(p, mc, d, f, X_own, X_slices[1:], X_land, G_up, True, rank),                    # dW_up = AG(X)^T G_up
    ]
    layers[0]["out"] = dict(O=layers[0]["out"]["O"], gathered=G_all)
    layers[3]["out"]["gathered"] = X_all
    return dict(layers=layers)


def _prepare_attn(c, mk, rank):
    p, B, h, S, n = c["p"], c["batch"], c["heads"], c["seq"], c["n"]
    mc, hd = B * S // p, h * HEAD_DIM
    Q, K, V = (mk.normal((B, h, S, HEAD_DIM)) for _ in range(3))
    Wo = mk.weight(hd, n, 0.02)
    stage = [mk.normal((mc, n), 0.02 * math.sqrt(hd * i / S), "f32") for i in range(1, p)]
    desc = cf.attn_desc(p, rank, B, h, S, HEAD_DIM, n, 1.0 / math.sqrt(HEAD_DIM))
    O = _out(mc, n)
    sends = [_out(mc, n) for _ in range(p - 1)]
    st = dict(desc=desc, args=(Q, K, V, Wo), stage=stage)
    if c["kind"] == "attn":
        scratch = _out(p * mc, hd, dtype=torch.bfloat16)
        each = [_out(mc, n) for _ in range(p - 1)]
        st["bufs"] = cf.make_attn_buffers(Q, K, V, Wo, scratch, O, stage, (None, None), (None, None), None, each, sends)
        st["keep"] = scratch
        st["out"] = dict(O=O, sent=sends, landed=each)
    else:
        st["scratch"] = _out(mc, hd, dtype=torch.bfloat16)
        st["recv"] = [None] + stage
        st["out"] = sends + [O]
    return st


def prepare(case, seed):
    _register_workspace()
    c, kind, p = case, case["kind"], case["p"]
    mk = _Maker(seed)
    rank = 1 % p
    if kind == "steps":
        st = _prepare_steps(c, mk, rank)
    elif kind in ("rs", "rs_pair"):
        A = mk.normal((p * c["m_chunk"], c["k"]))
        W = mk.weight(c["k"], c["n"], 0.02, c["layout"])
        st = dict(layers=[_rs_layer(mk, p, c["m_chunk"], c["n"], c["k"], A, W, 0.02, c["layout"], rank,
                                    cf.CF_KIND_RS if kind == "rs" else cf.CF_KIND_RS_PAIR, c.get("m", 1))])
    elif kind == "ag":
        slices = [mk.normal((c["m_chunk"], c["k"])) for _ in range(p)]
        each = [_out(c["m_chunk"], c["k"], dtype=torch.bfloat16) for _ in range(p - 1)]
        W = mk.weight(c["k"], c["n"], 0.02, c["layout"])
        st = dict(layers=[_ag_layer(mk, p, c["m_chunk"], c["n"], c["k"], slices[0], slices[1:], each, W, c["layout"], c["out"], rank,
                                    c.get("m", 1))])
    elif kind == "mlp":
        mc, d, f = c["m_chunk"], c["d"], c["f"]
        slices = [mk.normal((mc, d)) for _ in range(p)]
        each = [_out(mc, d, dtype=torch.bfloat16) for _ in range(p - 1)]
        up = _ag_layer(mk, p, mc, f, d, slices[0], slices[1:], each, mk.weight(d, f, 0.02), "kn", "bf16", rank)
        down = _rs_layer(mk, p, mc, d, f, up["out"]["O"], mk.weight(f, d, 0.02), 0.02, "kn", rank)
        st = dict(layers=[up, down])
    elif kind == "backward":
        st = _prepare_backward(c, mk, rank)
    elif kind in ("attn", "attn_steps"):
        st = _prepare_attn(c, mk, rank)
    else:
        bucket = mk.normal((p * c["chunk"],), 1e-3, "f32")
        stage = [mk.normal((c["chunk"],), 1e-3, "f32") for _ in range(p - 1)]
        each = [_out(c["chunk"]) for _ in range(p - 1)]
        desc = cf.layer_desc(p, rank, c["chunk"], 0, 0, "f32", "f32")
        bufs = cf.make_buffers(None, None, bucket, stage, (None, None), (None, None), None, each)
        st = dict(layers=[dict(desc=desc, kind=cf.CF_KIND_DP if kind == "dp" else cf.CF_KIND_DP_PAIR, bufs=bufs, keep=stage,
                               out=dict(bucket=bucket, landed=each))])
    st["case"] = kind if kind != "steps" else c["op"] + "_steps"
    return st


# ---------------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------------
def run(state):
    s = torch.cuda.current_stream()
    what = state["case"]
    if what == "rs_steps":
        call, desc, A, W = state["call"], state["desc"], state["A"], state["W"]
        for i, (recv, out) in enumerate(zip(state["recv"], state["out"])):
            call(desc, i, A, W, recv, out, s)
        return state["out"]
    if what == "ag_steps":
        desc, W, O = state["desc"], state["W"], state["out"]
        for i, shard in enumerate(state["slices"]):
            cf.ag_step(desc, i, shard, W, O, s)
        return O
    if what == "attn":
        cf.run_attn_schedule(state["desc"], state["bufs"], s, s, ONE_LAUNCH)
        return state["out"]
    if what == "attn_steps":
        desc, (Q, K, V, Wo), scratch = state["desc"], state["args"], state["scratch"]
        for i, (recv, out) in enumerate(zip(state["recv"], state["out"])):
            cf.attn_rs_step(desc, i, Q, K, V, Wo, recv, out, scratch, s)
        return state["out"]
    for layer in state["layers"]:
        cf.run_schedule(layer["desc"], layer["kind"], layer["bufs"], s, s, ONE_LAUNCH)
    return [layer["out"] for layer in state["layers"]]


def tolerance(case):
    """About four times the largest error seen against the same path in fp64 (2-norms), over the ranges above."""
    kind = case["kind"]
    if kind == "dp":
        return "exact"                       # one addition per element, whatever the order
    if kind == "dp_pair":
        return {"rel": 4e-7}                 # up to seven additions per element (seen: 1e-7)
    if kind in ("attn", "attn_steps"):
        return {"rel": 1e-2}                 # probabilities and attention output in bf16 (seen: 2.6e-3)
    if kind == "mlp" or (kind == "ag" and case["out"] == "bf16"):
        return {"rel": 5e-4}                 # bf16 activations: sums that round to the other neighbour (seen: 1.1e-4)
    return {"rel": 5e-6}                     # fp32 sums of up to 8192 products (seen: 6e-7, fp32 operands 1.1e-6)
