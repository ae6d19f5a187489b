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


@pytest.mark.parametrize("shape", ["1x4x1", "1x4x3", "2x4x1", "4x4x1"])
@pytest.mark.parametrize("rows,cols,off", [(1, 16, 0), (1, 24, 0), (3, 24, 0), (2, 40, 0), (3, 40, 8), (5, 32, 0), (8, 40, 0)])
def test_every_tile_of_whole_lines_is_computed_once(shape, rows, cols, off):
    """64 columns of [k x n] bf16 weights are a 128-byte line: from 24 tile columns on (rank steps: 40) these are dealt out one by
    one, and in bands where rows do not lie on the lines.  A step, and reduce-scatter and all-gather rank steps of four ranks."""
    mf, nc, ks = map(int, shape.split("x"))
    p, m, n, k = 4, rows * 16 * mf - 3, cols * 16 * nc, 1096
    g = torch.Generator(device=DEV).manual_seed(rows * 100 + cols + off)
    rnd = lambda *s: torch.empty(s, device=DEV).normal_(generator=g)
    nan = lambda *s: torch.full(s, float("nan"), device=DEV)
    A, W, B = rnd(p * m, k).bfloat16(), rnd(k, n + off).bfloat16()[:, :n], [rnd(m, n) for _ in range(p - 1)]
    slices = list(A.view(p, m, k).clone())
    out, sends, landed = nan(m, n), [nan(m, n) for _ in range(p - 1)], [nan(m, n) for _ in range(p - 1)]
    rs_out, ag_out, gathered = nan(m, n), nan(p * m, n), [torch.zeros_like(slices[0]) for _ in range(p - 1)]
    desc = cf.layer_desc(p, 1, m, n, k, ldw=n + off)
    rs = cf.make_buffers(A, W.data_ptr(), rs_out, B, (None, None), (None, None), None, landed, sends)
    ag = cf.make_buffers(slices[0], W.data_ptr(), ag_out, slices[1:], (None, None), (None, None), None, gathered)
    ws = torch.zeros(64 << 20, dtype=torch.uint8, device=DEV)
    os.environ["COMMFUSE_ROWS"] = shape
    try:
        cf.set_workspace(ws)
        torch.cuda.synchronize()
        cf.rs_step(cf.layer_desc(2, 0, m, n, k, ldw=n + off), 1, A, W.data_ptr(), B[0], out)
        for kind, bufs in ((cf.CF_KIND_RS, rs), (cf.CF_KIND_AG, ag)):
            cf.run_schedule(desc, kind, bufs, None, None, cf.CF_PERSISTENT | cf.CF_SERIAL | cf.CF_FUSED_COPY)
        torch.cuda.synchronize()
    finally:
        os.environ.pop("COMMFUSE_ROWS", None)
        cf.set_workspace(None)
    # sums of k products, a rounding of half an ulp of the running sum each
    close = lambda got, want: float((got.double() - want).abs().max() / want.abs().max()) <= 2.0 ** -24 * k ** 0.5 * 4
    full = A.double() @ W.double()
    product = lambda c: full[c * m:(c + 1) * m]
    assert close(out, product(0) + B[0].double())
    for i in range(p):
        c = (1 - i - 1) % p
        assert close(rs_out if i == p - 1 else sends[i], product(c) + (B[i - 1].double() if i else 0))
        assert close(ag_out[(1 - i) % p * m:((1 - i) % p + 1) * m], product(i))
    assert all(torch.equal(a, b) for a, b in zip(landed, B)) and all(torch.equal(a, b) for a, b in zip(gathered, slices[1:]))


@pytest.mark.parametrize("shape", ["1x1x1", "1x2x1", "2x4x1", "4x4x1", "1x2x3"])
@pytest.mark.parametrize("rows,n,k", [(1, 6144, 520), (3, 6656, 1096), (2, 6152, 1096), (1, 6144, 2056), (2, 6136, 264)])
def test_every_tile_of_wide_weights_is_computed_once(shape, rows, n, k):
    """[n x k] weights of 6144 rows and more over less than 2048 of k go one by one where their tiles come in eights."""
    mf, nc, ks = map(int, shape.split("x"))
    m = rows * 16 * mf - 3
    g = torch.Generator(device=DEV).manual_seed(rows * 100 + k)
    A = torch.empty(m, k, device=DEV).normal_(generator=g).bfloat16()
    W = torch.empty(n, k, device=DEV).normal_(generator=g).bfloat16()
    out = torch.full((m, n), float("nan"), device=DEV)
    ws = torch.zeros(64 << 20, dtype=torch.uint8, device=DEV)
    os.environ["COMMFUSE_ROWS"] = shape
    try:
        cf.set_workspace(ws)
        torch.cuda.synchronize()
        cf.ag_step(cf.layer_desc(1, 0, m, n, k, w_layout=cf.CF_W_NK), 0, A, W, out, None)
        torch.cuda.synchronize()
    finally:
        os.environ.pop("COMMFUSE_ROWS", None)
        cf.set_workspace(None)
    want = A.double() @ W.double().t()
    assert float((out.double() - want).abs().max() / want.abs().max()) <= 2.0 ** -24 * k ** 0.5 * 4
