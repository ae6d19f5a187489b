"""Tile kernels with the k range split over workgroups: the partial tiles, parked in the order the threads hold them, there and
back -- two to eight splits, tiles partly outside the matrix, every tile shape, fp32 and bf16 output, weight gradients in place."""
import os

import pytest
import torch

from paper_2604_24013_amd import binding as cf

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture
def split():
    def use(ks, tile, deep):
        os.environ.update(COMMFUSE_SPLITK=str(ks), COMMFUSE_TILE=tile, COMMFUSE_DEEP=deep)
    yield use
    for v in ("COMMFUSE_SPLITK", "COMMFUSE_TILE", "COMMFUSE_DEEP"):
        os.environ.pop(v, None)
    cf.set_workspace(None)


@pytest.mark.parametrize("ks", [2, 3, 8])
@pytest.mark.parametrize("tile,deep", [("128x128", "1"), ("128x128", "0"), ("256x128", "0"), ("256x256", "0")])
@pytest.mark.parametrize("m,n,k", [(130, 136, 1544), (256, 256, 1024), (1, 8, 520)])
def test_sums_of_the_splits(split, ks, tile, deep, m, n, k):
    g = torch.Generator(device=DEV).manual_seed(ks)
    rnd = lambda *s: torch.empty(s, device=DEV).normal_(generator=g)
    A, W, G, B, dW0 = rnd(m, k).bfloat16(), rnd(k, n).bfloat16(), rnd(k, m).bfloat16(), rnd(m, n), rnd(m, n)
    bm, bn = map(int, tile.split("x"))
    parts = ks * (-(-m // bm)) * (-(-n // bn)) * bm * bn * 4
    ws = torch.full(((64 << 10) + parts,), 0xFF, dtype=torch.uint8, device=DEV)          # to the byte: NaN partials, counters cleared below
    tol = 2.0 ** -24 * k ** 0.5 * 4                               # k roundings of half an ulp of the running sum
    split(ks, tile, deep)
    cf.set_workspace(ws)
    want, wgrad = A.double() @ W.double(), G.double().t() @ W.double()
    close = lambda got, ref, t: float((got.double() - ref).abs().max() / ref.abs().max()) <= t
    for _ in range(2):                                            # (the counters are zero again for the second pass)
        nan = lambda dtype: torch.full((m, n), float("nan"), dtype=dtype, device=DEV)
        rs, ag, ag16, dW = nan(torch.float32), nan(torch.float32), nan(torch.bfloat16), dW0.clone()
        torch.cuda.synchronize()
        cf.rs_step(cf.layer_desc(2, 0, m, n, k), 1, torch.cat([A, A]), W, B, rs)
        cf.ag_step(cf.layer_desc(1, 0, m, n, k), 0, A, W, ag)
        cf.ag_step(cf.layer_desc(1, 0, m, n, k, out_dtype="bf16"), 0, A, W, ag16)
        if m % 8 == 0:
            cf.wgrad_step(cf.layer_desc(2, 0, k, n, m), 1, G, W, dW)
        torch.cuda.synchronize()
        assert close(rs, want + B.double(), tol) and close(ag, want, tol) and close(ag16, want, tol + 2.0 ** -8)
        assert m % 8 or close(dW, wgrad + dW0.double(), tol)
    assert bool(torch.isfinite(ws[64 << 10:].view(torch.float32)).any()) == (-(-k // 64) > 1)   # the splits did meet there
    cf.set_workspace(ws[:-16])                                    # sixteen bytes short: unsplit, the workspace untouched
    ws[64 << 10:] = 0xFF
    torch.cuda.synchronize()
    cf.rs_step(cf.layer_desc(2, 0, m, n, k), 1, torch.cat([A, A]), W, B, rs)
    torch.cuda.synchronize()
    full = min(ks, -(-k // 64)) == ks
    assert close(rs, want + B.double(), tol) and (not full or bool((ws[64 << 10:] == 0xFF).all()))
