"""The few-rows kernel deals its tiles out in a band of columns per XCD: grids of fewer tiles than XCDs, of whole octets and one off
them, one and several row tiles, k ranges split over workgroups.  Every element of every output, against the product in 64 bits."""
import os

import pytest
import torch

from paper_2604_24013_amd import binding as cf

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("shape", ["1x2x1", "2x4x1", "4x4x1", "1x2x3"])
@pytest.mark.parametrize("rows,cols", [(1, 1), (1, 7), (1, 8), (1, 9), (3, 3), (2, 8), (5, 13), (33, 1)])
def test_every_tile_is_computed_once(shape, rows, cols):
    mf, nc, ks = map(int, shape.split("x"))
    m, n, k = rows * 16 * mf - 3, cols * 16 * nc - 8, 1544
    g = torch.Generator(device=DEV).manual_seed(rows * 100 + cols)
    A = torch.empty(m, k, device=DEV).normal_(generator=g).bfloat16()
    W = torch.empty(k, n, device=DEV).normal_(generator=g).bfloat16()
    B = torch.empty(m, n, device=DEV).normal_(generator=g)
    ws = torch.zeros(64 << 20, dtype=torch.uint8, device=DEV)
    out = torch.full((m, n), float("nan"), device=DEV)
    os.environ["COMMFUSE_ROWS"] = shape
    try:
        cf.set_workspace(ws)
        torch.cuda.synchronize()
        cf.rs_step(cf.layer_desc(2, 0, m, n, k), 1, torch.cat([A, A]), W, B, out, None)
        torch.cuda.synchronize()
    finally:
        os.environ.pop("COMMFUSE_ROWS", None)
        cf.set_workspace(None)
    want = A.double() @ W.double() + B.double()
    # sums of k products, a rounding of half an ulp of the running sum each
    assert float((out.double() - want).abs().max() / want.abs().max()) <= 2.0 ** -24 * k ** 0.5 * 4
