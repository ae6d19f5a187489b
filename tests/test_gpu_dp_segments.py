"""All adds of a ring gradient reduce in one launch: slice lengths around the vectors, the chunks and the rules of the launch
(8M elements: one-wave workgroups; 1.5M: two vectors per lane in the pairwise sum), slices off the 16-byte grid; every element bit for bit (one fp32 addition each)."""
import numpy as np
import pytest
import torch

from paper_2604_24013_amd import binding as cf
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("carry", [0, cf.CF_FUSED_COPY])
@pytest.mark.parametrize("p,m,c", [(2, 1, 1), (8, 1, 3), (4, 2, 8), (8, 2, 4094), (3, 1, 4095), (8, 1, 4096), (8, 1, 4097), (2, 1, 12289),
                                   (2, 1, (8 << 20) - 1), (2, 1, 8 << 20), (3, 1, (8 << 20) + 5), (4, 1, (3 << 19) - 1), (4, 1, 3 << 19)])
def test_ring_and_pairwise_in_one_launch(p, m, c, carry):
    rng = np.random.default_rng(c)
    g = rng.standard_normal(p * c, dtype=np.float32)
    R = [rng.standard_normal(c, dtype=np.float32) for _ in range(p - 1)]
    for kind in (cf.CF_KIND_DP, cf.CF_KIND_DP_PAIR):
        if kind == cf.CF_KIND_DP_PAIR and (p % 2 or m > 1):
            continue
        want = g.copy()
        rank = p - 1
        for i in range(1, p):
            l = cf.chunk_index(cf.CF_KIND_DP, p, rank, i) if kind == cf.CF_KIND_DP else rank
            want[l * c:(l + 1) * c] = R[i - 1] + want[l * c:(l + 1) * c]
        bucket = torch.from_numpy(g.copy()).to(H.DEV)
        stage = [torch.from_numpy(r).to(H.DEV) for r in R]
        each = [torch.full((c,), float("nan"), device=H.DEV) for _ in R]
        desc = cf.layer_desc(p, rank, c, 0, 0, "f32", "f32", m=m)
        bufs = cf.make_buffers(None, None, bucket, stage, (None, None), (None, None), None, each)
        st = torch.cuda.Stream()
        torch.cuda.synchronize()
        cf.run_schedule(desc, kind, bufs, st, st, cf.CF_PERSISTENT | cf.CF_SERIAL | carry)
        st.synchronize()
        assert np.array_equal(bucket.cpu().numpy(), want), kind
        assert all(torch.equal(a, b) for a, b in zip(each, stage)), kind
