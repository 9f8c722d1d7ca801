"""Attention where its schedule changes: items run whole (11 key tiles) or cut (12), little work on
a few shares, cut items at head dim 16, 64 and 128, ragged last key tiles, the merge pass over more
requests than it walks."""
import numpy as np
import pytest
import torch

from paper_2607_12121_amd import flashdiff as fdl
from paper_2607_12121_amd import workloads as wl
from tests import gpu_harness as gh
from tests.helpers import small_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    fdl.lib()


@pytest.mark.parametrize("dh,H", [(16, 4), (64, 2), (128, 1)])
@pytest.mark.parametrize("sizes,active", [((704,), 2), ((705,), 2), ((2048,), 1), ((1024, 65, 3000), 2), ((2048, 33), 40),
                                          ((1500,) + (70,) * 19, 1)])
def test_attention_schedule_edges(dh, H, sizes, active):
    """`active` 32-token regions of each request (all of them where it has fewer)."""
    D = max(64, H * dh)
    w = small_workload("audio", requests=tuple(wl.RequestShape("seq", (n,), (32,)) for n in sizes), activity="frac",
                       activity_args=(0.5, 0.5), L=1, D=D, H=D // dh, dh=dh, F=128)
    case = gh.make_case("audio", workload=w)
    # only the hot regions move, so that exactly the first `active` regions of a request run
    off = case.rmap.req_reg_off
    x_prev = case.inp.x_prev.copy()
    x_cur = x_prev.copy()
    eps = np.zeros(len(sizes))
    for b in range(len(sizes)):
        regions = np.arange(off[b], off[b + 1])
        hot = regions[:active]
        x_cur[np.isin(case.rmap.token_region, hot)] += 1.0
        eps[b] = 0.5 / len(hot) if len(hot) < len(regions) else 0.0
    gh.say(f"attention schedule edges dh={dh} sizes={sizes[:3]} n={len(sizes)} active={active}")
    g, st = gh.run_gpu(case, eps, x_cur, x_prev)
    assert g["M"] == sum(min(n, 32 * active) for n in sizes)
    o = gh.run_oracle(case, eps, x_cur, x_prev)
    gh.compare_step(case, g, o, x_cur, st)
