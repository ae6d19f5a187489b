"""Weight gradients whose launch takes the moving operand from the neighbours' buffers and lands it: dW and the gathered buffer are
bit for bit those of the copies in front."""
import pytest
import torch

from paper_2604_24013_amd import binding as cf
from paper_2604_24013_amd import emulated_rank as H

pytestmark = pytest.mark.gpu

COPIED = cf.CF_PERSISTENT | cf.CF_SERIAL
CARRIED = COPIED | cf.CF_FUSED_COPY


@pytest.mark.parametrize("left_moves", [True, False])
@pytest.mark.parametrize("p,mc,m,k,n", [
    (2, 128, 1, 256, 256),                   # two k-tiles to a block, one work item that lands them all
    (2, 192, 1, 256, 2048), (3, 192, 1, 2048, 256),              # more work items side by side than k-tiles; an odd number of k-tiles to a block
    (15, 128, 1, 512, 768),                  # as many blocks as a launch has room for
    (4, 256, 2, 768, 512),                   # two sub-steps to a hop
    (2, 128, 1, 4864, 4096),                 # 304 work items: a second round
    (2, 64, 1, 256, 256), (2, 96, 1, 256, 256), (2, 128, 1, 256, 264),   # copied in front: one k-tile to a block, ragged ones, ragged columns
])
def test_carried_deliveries_change_nothing(monkeypatch, left_moves, p, mc, m, k, n):
    monkeypatch.setenv("COMMFUSE_TILE", "256x256")
    g = torch.Generator().manual_seed(p * mc + k + n)
    rnd = lambda rows, cols: torch.empty(rows, cols).normal_(generator=g).bfloat16().view(torch.int16).numpy().view("uint16")
    moving, local = [rnd(mc, k if left_moves else n) for _ in range(p)], rnd(p * mc, n if left_moves else k)
    for rank in sorted({0, p // 2, p - 1}):
        got = []
        for flags in (COPIED, CARRIED, CARRIED | cf.CF_GRAPH):
            run = H.WgradRun(p, rank, mc, k, n, moving, local, left_moves, m=m, gathered=True)
            for _ in range(2 if flags & cf.CF_GRAPH else 1):
                run.dW.fill_(float("nan"))
                for each in run.each:
                    each.fill_(float("nan"))
                run.run_schedule(flags)
            got.append((run.dW, run.gathered.view(torch.int16)))
        for dW, gathered in got[1:]:
            assert not bool(dW.isnan().any()) and torch.equal(dW, got[0][0]) and torch.equal(gathered, got[0][1])
