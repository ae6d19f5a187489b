"""The one-launch reduce-scatter's epilogue: B_in read once in whole lines, landed and added from the same registers.

Every tile shape, at remainders of rows, columns and k-tiles, carried against copied: landing buffers byte for byte, sums bit
for bit, and against the product in 64 bits."""
import os

import pytest
import torch

from paper_2604_24013_amd import binding as cf
from paper_2604_24013_amd import emulated_rank as H

pytestmark = pytest.mark.gpu

ONE_LAUNCH = cf.CF_PERSISTENT | cf.CF_SERIAL
DEV = "cuda:0"


def _run(p, mc, n, k, layout, ldo, flags, seed=5):
    g = torch.Generator(device=DEV).manual_seed(seed)
    rnd = lambda *s: torch.empty(s, device=DEV).normal_(generator=g)
    nan = lambda: torch.full((mc, ldo), float("nan"), device=DEV)
    A, W = rnd(p * mc, k).bfloat16(), rnd(*((k, n) if layout == cf.CF_W_KN else (n, k))).bfloat16()
    stage = [rnd(mc, ldo) for _ in range(p - 1)]
    O, each, sends = nan(), [nan() for _ in range(p - 1)], [nan() for _ in range(p - 1)]
    bufs = cf.make_buffers(A, W, O, stage, (None, None), (None, None), None, each, sends)
    desc = cf.layer_desc(p, 1 % p, mc, n, k, "bf16", "f32", layout, ldo=ldo)
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    cf.run_schedule(desc, cf.CF_KIND_RS, bufs, st, st, ONE_LAUNCH | flags)
    st.synchronize()
    return A, W if layout == cf.CF_W_KN else W.t(), stage, each, sends + [O]


@pytest.mark.parametrize("tile,deep", [("256x256", "0"), ("256x128", "0"), ("128x128", "0"), ("128x128", "1")])
@pytest.mark.parametrize("layout", [cf.CF_W_KN, cf.CF_W_NK])
@pytest.mark.parametrize("p,mc,n,k,pad", [
    (4, 256, 512, 64, 0),        # whole tiles, one k-tile: the early request of B_in follows the prologue
    (4, 256, 256, 128, 0), (3, 256, 256, 192, 0), (2, 130, 264, 256, 0), (2, 256, 128, 320, 0),   # two to five k-tiles: the iterations without loads
    (8, 512, 256, 1152, 0),      # whole tiles, eighteen k-tiles
    (3, 261, 264, 136, 0),       # a tile of five rows and of eight columns, a ragged third k-tile; rows off the 128-byte lines
    (2, 130, 264, 3080, 0),      # forty-nine k-tiles: two 128x128 tiles per compute unit issue their loads in a burst
    (2, 1, 8, 8, 0),             # one row, two chunks of columns
    (2, 200, 232, 1288, 24),     # padded rows, twenty-one k-tiles: carried on 256x256 tiles, else copied with the padding
    (3, 261, 264, 1152, 8),      # ... eighteen whole k-tiles, a second tile row of five rows
    (8, 512, 1024, 1280, 64),    # ... whole tiles
    (2, 200, 232, 1160, 24),     # ... nineteen with a ragged last one: copied
    (2, 130, 96, 200, 32),       # padded rows, few k-tiles: copied
    (8, 1024, 2048, 328, 0),     # work items for every compute unit of any tile: half of them land in front of the main loop
    (4, 1000, 4096, 72, 0),      # likewise, tiles partly outside the matrix
])
def test_carried_sums_and_landings_are_the_copied_ones(tile, deep, layout, p, mc, n, k, pad):
    os.environ["COMMFUSE_TILE"], os.environ["COMMFUSE_DEEP"] = tile, deep
    try:
        A, W, stage, each, outs = _run(p, mc, n, k, layout, n + pad, cf.CF_FUSED_COPY)
        _, _, _, _, copied = _run(p, mc, n, k, layout, n + pad, 0)
    finally:
        os.environ.pop("COMMFUSE_TILE", None)
        os.environ.pop("COMMFUSE_DEEP", None)
    for a, b in zip(each, stage):
        assert torch.equal(a[:, :n], b[:, :n])
        if pad and tile == "256x256" and (k + 63) // 64 >= (20 if k % 64 else 18):
            assert bool(a[:, n:].isnan().all())      # carried: without the padding
        else:
            assert torch.equal(a, b)                 # a copy in front moves the padding too
    for i, (got, same) in enumerate(zip(outs, copied)):
        assert torch.equal(got[:, :n], same[:, :n])
        assert bool(got[:, n:].isnan().all())
        l = cf.chunk_index(cf.CF_KIND_RS, p, 1 % p, i)
        want = A[l * mc:(l + 1) * mc].double() @ W.double() + (stage[i - 1][:, :n].double() if i else 0.0)
        # fp32 sums of k products of unit variance: k roundings of 2^-24 at sqrt(k) on average, four times that at most
        assert H.rel_err(H.to_host_f64(got[:, :n]), H.to_host_f64(want)) <= 4 * k ** 0.5 * 2.0 ** -24 + 1e-6
