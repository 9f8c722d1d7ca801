"""Attention where its schedule changes: items run whole or cut, little work on a few shares, cut
items at head dim 16, 64 and 128, ragged last key tiles, the merge pass over more requests than it
walks, more items than workgroups."""
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


def _run(dh, H, sizes, active):
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
    gh.say(f"attention schedule edges dh={dh} H={H} sizes={sizes[:3]} n={len(sizes)} active={active}")
    g, st = gh.run_gpu(case, eps, x_cur, x_prev)
    assert g["M"] == sum(min(n, 32 * active) for n in sizes)
    o = gh.run_oracle(case, eps, x_cur, x_prev)
    gh.compare_step(case, g, o, x_cur, st)


@pytest.mark.parametrize("dh,H", [(16, 4), (64, 2), (128, 1)])
@pytest.mark.parametrize("sizes,active", [((704,), 2), ((705,), 2), ((2048,), 1), ((1024, 65, 3000), 2), ((2048, 33), 40),
                                          ((1500,) + (70,) * 19, 1)])
def test_attention_schedule_edges(dh, H, sizes, active):
    _run(dh, H, sizes, active)


@pytest.mark.parametrize("dh,H,sizes,active", [
    (128, 1, (768,), 2), (128, 1, (769,), 2),            # the last size without the merge's launch, the first that cuts
    (128, 1, (16384,), 2), (128, 1, (16385,), 2),        # cut items at any length
    (128, 4, (3000,) + (70,) * 70, 1),                   # 284 items on 256 workgroups, mixed: cut
    (128, 4, (130,) * 66, 5),                            # 264 items of one length: whole rounds
    (64, 16, (1024,) * 4, 32),                           # 256 items of one length: whole, the merge finds nothing
])
def test_attention_cut_rule(dh, H, sizes, active):
    """Both sides of the rule that cuts items, with items for every workgroup no more than once and
    with more of them."""
    _run(dh, H, sizes, active)
