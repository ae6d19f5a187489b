"""What a call enqueues -- which kernels, in which grid, and which copies -- read off the library's host code without a GPU."""
import os

import pytest

from paper_2604_24013_amd import binding as cf
from tests.dry import Dry

ONE_LAUNCH = cf.CF_PERSISTENT | cf.CF_SERIAL


def P(i):
    return (i + 1) << 33                              # fake, aligned, far apart


@pytest.fixture(scope="module")
def dry(tmp_path_factory):
    return Dry(str(tmp_path_factory.mktemp("dry")))


@pytest.mark.parametrize("cus", [32, 64, 256])
def test_grids_follow_the_devices_compute_units(dry, monkeypatch, cus):
    monkeypatch.setenv("COMMFUSE_DRY_CUS", str(cus))
    step = cf.layer_desc(1, 0, 4096, 8192, 1024)
    calls = [lambda: cf.ag_step(step, 0, P(0), P(1), P(2)), lambda: cf.rs_step(cf.layer_desc(2, 0, 4096, 8192, 1024), 1, P(0), P(1), P(2), P(3)),
             lambda: cf.wgrad_step(cf.layer_desc(1, 0, 1024, 8192, 4096), 0, P(0), P(1), P(2)),
             lambda: cf.run_schedule(cf.layer_desc(2, 0, 4096, 8192, 1024), cf.CF_KIND_AG,
                                     cf.make_buffers(P(0), P(1), P(2), [P(3)], (None, None), recv_each=[P(4)]), None, None,
                                     ONE_LAUNCH | cf.CF_FUSED_COPY)]
    for call in calls:
        (kernel, grid, block), = dry.calls(call)
        assert kernel.startswith("gemm_bf16_dl_kernel<256, 256,") and (grid, block) == (cus, 512)
