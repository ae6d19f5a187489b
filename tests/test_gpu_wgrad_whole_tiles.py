"""Weight-gradient GEMMs on whole tiles: the left operand stored by k-rows on the 16x16x32 main loop, against 64 bits."""
import os

import pytest
import torch

from paper_2604_24013_amd import binding as cf
from paper_2604_24013_amd import emulated_rank as H

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("tile", ["256x256", "256x128", "128x128"])
@pytest.mark.parametrize("mc,k,n,pad", [
    (64, 256, 256, 0), (128, 256, 512, 0), (192, 512, 256, 0),   # one to three k-tiles: no steady state
    (8, 256, 256, 0), (72, 256, 256, 8), (1000, 512, 768, 0),    # a ragged last k-tile, alone and behind whole ones
    (1024, 256, 2048, 64),                                       # eight tile columns: a band for each XCD; padded rows
    (320, 4864, 4096, 0),                                        # 304 work items of 256x256: a second round
    (136, 264, 520, 0),                                          # rows and columns outside the matrix
])
def test_wgrad_steps_accumulate_in_place(tile, mc, k, n, pad):
    g = torch.Generator(device=DEV).manual_seed(mc + k)
    rnd = lambda *s: torch.empty(s, device=DEV).normal_(generator=g).bfloat16()
    p = 2
    left, right = [rnd(mc, k + pad) for _ in range(p)], [rnd(mc, n + pad) for _ in range(p)]
    dW = torch.full((k, n + pad), float("nan"), device=DEV)
    desc = cf.layer_desc(p, 1, mc, n, k, "bf16", "f32", lda=k + pad, ldw=n + pad, ldo=n + pad)
    want = torch.zeros((k, n), dtype=torch.float64, device=DEV)
    os.environ["COMMFUSE_TILE"] = tile
    try:
        for i in range(p):
            cf.wgrad_step(desc, i, left[i], right[i], dW, torch.cuda.current_stream())
            want += left[i][:, :k].t().double() @ right[i][:, :n].double()
            # fp32 sums of (i + 1) mc products of unit variance: as many roundings of 2^-24, four times their square root at most
            assert H.rel_err(H.to_host_f64(dW[:, :n]), H.to_host_f64(want)) <= 4 * ((i + 1) * mc) ** 0.5 * 2.0 ** -24 + 1e-6
            assert bool(dW[:, n:].isnan().all())
    finally:
        os.environ.pop("COMMFUSE_TILE", None)
