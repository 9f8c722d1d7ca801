"""Region importance at the edges of its 32-row tiles: regions of 1, 31, 32, 33 and
257 tokens (ragged last tiles of keys and queries, more tiles than waves), head dims
16, 64 and 128, one and several requests."""
import numpy as np
import pytest
import torch

from paper_2607_12121_amd import flashdiff as fdl
from paper_2607_12121_amd import workloads as wl
from tests import gpu_harness as gh
from tests.helpers import rel_err, small_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    fdl.lib()


@pytest.mark.parametrize("dh,H", [(16, 4), (64, 2), (128, 1)])
@pytest.mark.parametrize("sizes,region", [((1, 5), 1), ((62, 40), 31), ((96,), 32), ((100, 33), 33), ((600, 257), 257)])
def test_importance_tile_edges(dh, H, sizes, region):
    D = max(64, H * dh)
    w = small_workload("audio", requests=tuple(wl.RequestShape("seq", (n,), (region,)) for n in sizes), activity="frac",
                       activity_args=(0.6, 1.0), L=1, D=D, H=D // dh, dh=dh, F=128)
    case = gh.make_case("audio", workload=w)
    gh.say(f"importance edges dh={dh} sizes={sizes} region={region}")
    g, st = gh.run_gpu(case, case.inp.eps, case.inp.x_cur, case.inp.x_prev, importance_block=0)
    o = gh.run_oracle(case, case.inp.eps, case.inp.x_cur, case.inp.x_prev, importance_block=0)
    gh.compare_step(case, g, o, case.inp.x_cur, st)
    act = g["active"]
    assert act.any()
    assert rel_err(g["importance"][act], o["importance"][act]) <= gh.TOL
    assert np.all(np.isnan(g["importance"][~act]))
