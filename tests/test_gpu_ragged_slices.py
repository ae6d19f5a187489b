"""The one-launch all-gather over a k range that is no multiple of the k-tile, its deliveries carried: landing buffers byte for
byte, the product bit for bit that of the copied mode and against 64 bits, on every tile shape."""
import os

import pytest
import torch

from paper_2604_24013_amd import binding as cf

pytestmark = pytest.mark.gpu

ONE_LAUNCH = cf.CF_PERSISTENT | cf.CF_SERIAL
DEV = "cuda:0"


def _run(p, mc, n, k, layout, m, out, flags, off=0):
    g = torch.Generator(device=DEV).manual_seed(3)
    rnd = lambda *s: torch.empty(s, device=DEV).normal_(generator=g).bfloat16()
    def at(t):                                                # `off` elements into its buffer
        b = torch.empty(t.numel() + off, dtype=t.dtype, device=DEV)[off:].view(t.shape)
        return b.copy_(t)
    slices, W = [rnd(mc, k)] + [at(rnd(mc, k)) for _ in range(p - 1)], rnd(*((k, n) if layout == cf.CF_W_KN else (n, k)))
    each = [at(torch.full((mc, k), float("nan"), dtype=torch.bfloat16, device=DEV)) for _ in range(p - 1)]
    O = torch.full((p * mc, n), float("nan"), dtype=out, device=DEV)
    bufs = cf.make_buffers(slices[0], W, O, slices[1:], (None, None), (None, None), None, each)
    desc = cf.layer_desc(p, 1 % p, mc, n, k, "bf16", "bf16" if out == torch.bfloat16 else "f32", layout, m=m)
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    cf.run_schedule(desc, cf.CF_KIND_AG, bufs, st, st, ONE_LAUNCH | flags)
    st.synchronize()
    return slices, W if layout == cf.CF_W_KN else W.t(), each, O


@pytest.mark.parametrize("tile,deep", [("256x256", "0"), ("256x128", "0"), ("128x128", "0"), ("128x128", "1")])
@pytest.mark.parametrize("layout", [cf.CF_W_KN, cf.CF_W_NK])
@pytest.mark.parametrize("p,mc,n,k,m", [
    (3, 130, 264, 8, 1),         # one k-tile of one chunk
    (4, 256, 512, 120, 1),       # whole 256x256 tiles, a ragged second k-tile of seven chunks
    (2, 261, 1032, 200, 1),      # more tile columns than k-tiles: most carry nothing
    (2, 264, 136, 328, 2),       # one tile column carries every k-tile; sub-steps
    (8, 1, 8, 1096, 1),          # one row
    (2, 200, 264, 3208, 1),      # fifty-one k-tiles: two 128x128 tiles per compute unit issue their loads in a burst
])
def test_ragged_slices_land_whole(tile, deep, layout, p, mc, n, k, m):
    os.environ["COMMFUSE_TILE"], os.environ["COMMFUSE_DEEP"] = tile, deep
    out = torch.bfloat16 if (n // 8) % 2 else torch.float32
    try:
        slices, W, each, O = _run(p, mc, n, k, layout, m, out, cf.CF_FUSED_COPY)
        _, _, _, copied = _run(p, mc, n, k, layout, m, out, 0)
        _, _, apart, moved = _run(p, mc, n, k, layout, m, out, cf.CF_FUSED_COPY, off=4)     # off the 16-byte grid: copied in front
    finally:
        os.environ.pop("COMMFUSE_TILE", None)
        os.environ.pop("COMMFUSE_DEEP", None)
    assert all(torch.equal(a, b) for a, b in zip(each, slices[1:])) and all(torch.equal(a, b) for a, b in zip(apart, slices[1:]))
    assert torch.equal(O, copied) and torch.equal(O, moved)
    for i, s in enumerate(slices):
        want = s.double() @ W.double()
        c = (1 % p - i) % p
        got = O[c * mc:(c + 1) * mc].double()
        # fp32 sums of k products: k roundings of at most half an ulp of the running sum; bf16 results round once more
        tol = 2.0 ** -24 * k ** 0.5 * 4 + (2.0 ** -8 if out == torch.bfloat16 else 0)
        assert float((got - want).abs().max() / want.abs().max()) <= tol


@pytest.mark.parametrize("p,mc,n,k", [(4, 272, 1032, 264), (8, 130, 1536, 1096), (8, 8, 1536, 4104)])      # tiles; few rows
def test_two_streams_keep_the_copy_streams_order(p, mc, n, k):
    """What is enqueued on the copy stream before the call is read by it, and what is enqueued there after the call finds the
    deliveries landed and may overwrite the peers' buffers: the compute stream is busy for longer than that takes."""
    g = torch.Generator(device=DEV).manual_seed(5)
    rnd = lambda *s: torch.empty(s, device=DEV).normal_(generator=g).bfloat16()
    fresh, W = [rnd(mc, k) for _ in range(p)], rnd(k, n)
    nan = lambda t: torch.full_like(t, float("nan"))
    stage, each, O = [nan(t) for t in fresh[1:]], [nan(t) for t in fresh[1:]], torch.full((p * mc, n), float("nan"), device=DEV)
    bufs = cf.make_buffers(fresh[0], W, O, stage, (None, None), (None, None), None, each)
    cs, xs = torch.cuda.Stream(), torch.cuda.Stream()
    busy = torch.zeros(1 << 28, device=DEV)                          # a pass over it takes longer than the whole rank step
    torch.cuda.synchronize()
    with torch.cuda.stream(xs):
        for t, f in zip(stage, fresh[1:]):
            t.copy_(f)
    with torch.cuda.stream(cs):
        for _ in range(4):
            busy.add_(1.0)
    cf.run_schedule(cf.layer_desc(p, 1, mc, n, k), cf.CF_KIND_AG, bufs, cs, xs, cf.CF_PERSISTENT | cf.CF_FUSED_COPY)
    with torch.cuda.stream(xs):
        landed = [t.clone() for t in each]
        for t in stage:
            t.fill_(float("nan"))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(landed, fresh[1:]))
    for i, s in enumerate(fresh):
        want = s.double() @ W.double()
        c = (1 - i) % p
        assert float((O[c * mc:(c + 1) * mc].double() - want).abs().max() / want.abs().max()) <= 2.0 ** -24 * k ** 0.5 * 4
