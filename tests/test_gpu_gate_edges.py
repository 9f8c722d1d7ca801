"""Gate-side kernels at the sizes where their split changes: the index list around
one workgroup's chunk and the one-kernel limit (requests that start inside a chunk,
one request over several chunks, no active region), the one-pass and the cut region
score, and the cached-drift update in one launch."""
import numpy as np
import pytest
import torch

from oracle import flashdiff_oracle as orc
from paper_2607_12121_amd import flashdiff as fdl
from tests import gpu_harness as gh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    fdl.lib()


def _layout(rng, sizes, regions):
    """Requests of `sizes` tokens, each cut at random into `regions` regions."""
    maps, off, r0 = [], [0], 0
    for n in sizes:
        k = min(regions, n)
        m = np.concatenate([np.arange(k), rng.integers(0, k, n - k)])
        rng.shuffle(m)
        maps.append(m + r0)
        r0 += k
        off.append(off[-1] + n)
    return orc.Layout(np.concatenate(maps), np.asarray(off), r0)


@pytest.mark.parametrize("sizes,regions", [([4096], 16), ([4097], 16), ([8192], 7), ([8193], 7), ([12289], 33),
                                           ([1, 4095, 4097, 63], 5), ([3000, 9000, 50, 5000], 64), ([9] * 1000, 2)])
@pytest.mark.parametrize("frac", [0.0, 0.4, 1.0])
def test_index_list_at_chunk_edges(sizes, regions, frac):
    rng = np.random.default_rng([len(sizes), sizes[0], regions])
    lay = _layout(rng, sizes, regions)
    N, R, B = len(lay.token_region), lay.n_regions, lay.n_requests
    gh.say(f"select N={N} R={R} B={B} frac={frac}")
    plan = fdl.make_plan(lay.token_region.astype(np.int32), lay.req_tok_off.astype(np.int32), R)
    score = (rng.random(R) < frac).astype(float)   # eps D <= 1: exactly the regions of score 1 run
    eps = np.full(B, 1e-6) if frac else np.full(B, np.inf)
    st, run = torch.zeros(R, dtype=torch.float64, device="cuda"), torch.zeros(R, dtype=torch.int32, device="cuda")
    act = torch.ones(R, dtype=torch.uint8, device="cuda")
    idx = torch.full((N,), -7, dtype=torch.int32, device="cuda")
    cu, m = torch.zeros(B + 1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    fdl.fd_select(plan, torch.from_numpy(score).cuda(), torch.from_numpy(eps).cuda(), 0.0, 0, st, run, act, act, idx,
                  cu, m)
    torch.cuda.synchronize()
    _, orun, oact = orc.gate_select(lay, score, np.zeros(R), np.zeros(R, np.int32), np.ones(R, bool), eps, 0.0, 0)
    oidx, ocu = orc.active_rows(lay, oact)
    np.testing.assert_array_equal(act.cpu().numpy().astype(bool), oact)
    np.testing.assert_array_equal(run.cpu().numpy(), orun)
    np.testing.assert_array_equal(cu.cpu().numpy(), ocu)
    assert int(m.item()) == len(oidx)
    np.testing.assert_array_equal(idx[:len(oidx)].cpu().numpy(), oidx)
    assert (idx[len(oidx):].cpu().numpy() == -7).all()


@pytest.mark.parametrize("C,size", [(16, 1), (64, 16), (64, 17), (64, 1024), (64, 1025), (256, 256), (256, 257), (48, 1365)])
def test_score_one_pass_and_cut(C, size):
    """Regions of two requests around the sizes at which the workgroup widens and a region is cut."""
    rng = np.random.default_rng([C, size])
    lay = _layout(rng, [3 * size, size + 1], 2)
    N, R = len(lay.token_region), lay.n_regions
    gh.say(f"score C={C} N={N}")
    plan = fdl.make_plan(lay.token_region.astype(np.int32), lay.req_tok_off.astype(np.int32), R)
    x, xp = (rng.standard_normal((N, C), dtype=np.float32) for _ in range(2))
    score = torch.zeros(R, dtype=torch.float64, device="cuda")
    ws = torch.empty(max(fdl.fd_region_score_ws_size(plan, C), 256), dtype=torch.uint8, device="cuda")
    fdl.fd_region_score(plan, C, torch.from_numpy(x).cuda(), torch.from_numpy(xp).cuda(), score, ws)
    # fp64 sums of non-negative terms in another order: at most (terms) * 2^-53 relative
    np.testing.assert_allclose(score.cpu().numpy(), orc.region_score(lay, x, xp), rtol=N * C * 2.0 ** -53, atol=0)


@pytest.mark.parametrize("C,R,size", [(64, 3, 128), (64, 3, 129), (64, 128, 256), (64, 127, 256), (64, 192, 1024), (64, 191, 1024),
                                      (256, 1, 256), (16, 5, 4097), (64, 2, 1025)])
def test_score_on_both_sides_of_the_pass_rule(C, R, size):
    """R regions of exactly `size` tokens, one pass or cut, through both entry points: the cut ones
    sum their partials in the caller's workspace and in the built-in scratch."""
    rng = np.random.default_rng([C, R, size])
    N = R * size
    region = np.arange(N) // size
    lay = orc.Layout(region, np.array([0, N]), R)
    gh.say(f"score pass rule C={C} R={R} size={size}")
    plan = fdl.make_plan(region.astype(np.int32), np.array([0, N], np.int32), R)
    x, xp = (rng.standard_normal((N, C), dtype=np.float32) for _ in range(2))
    dx, dxp = torch.from_numpy(x).cuda(), torch.from_numpy(xp).cuda()
    got, own = (torch.full((R,), np.nan, dtype=torch.float64, device="cuda") for _ in range(2))
    ws = torch.empty(max(fdl.fd_region_score_ws_size(plan, C), 256), dtype=torch.uint8, device="cuda")
    fdl.fd_region_score(plan, C, dx, dxp, got, ws)
    fdl.fd_region_score_noalloc(plan, C, dx, dxp, own)
    # fp64 sums of size * C non-negative terms in another order
    np.testing.assert_allclose(got.cpu().numpy(), orc.region_score(lay, x, xp), rtol=size * C * 2.0 ** -53, atol=0)
    assert torch.equal(got, own)


@pytest.mark.parametrize("C,sizes", [(16, [5]), (64, [127, 1, 130]), (48, [33, 700]), (256, [3, 2, 1])])
def test_drift_update_odd_sizes(C, sizes):
    rng = np.random.default_rng([C, len(sizes)])
    lay = _layout(rng, sizes, 3)
    N, R, B = len(lay.token_region), lay.n_regions, lay.n_requests
    gh.say(f"drift update C={C} N={N}")
    plan = fdl.make_plan(lay.token_region.astype(np.int32), lay.req_tok_off.astype(np.int32), R)
    act = rng.random(R) < 0.5
    idx, _ = orc.active_rows(lay, act)
    x, v, vc = (rng.standard_normal((N, C), dtype=np.float32) for _ in range(3))
    dt = rng.uniform(-0.1, 0.1, B).astype(np.float32)
    d_x, d_vc = torch.from_numpy(x).cuda(), torch.from_numpy(vc).cuda()
    d_idx = torch.zeros(N, dtype=torch.int32, device="cuda")
    d_idx[:len(idx)] = torch.from_numpy(idx.astype(np.int32)).cuda()
    m = torch.tensor([len(idx)], dtype=torch.int32, device="cuda")
    fdl.fd_scatter_update(plan, C, d_x, torch.from_numpy(v).cuda(), d_idx, m, torch.from_numpy(dt).cuda(), d_vc,
                          torch.from_numpy(act.astype(np.uint8)).cuda(), fdl.FD_SKIP_REUSE_DRIFT)
    drift = vc.copy()
    drift[idx] = v[:len(idx)]
    want = x + (dt[lay.token_request()][:, None] * drift).astype(np.float32)   # two fp32 roundings
    np.testing.assert_array_equal(d_x.cpu().numpy(), want)
    np.testing.assert_array_equal(d_vc.cpu().numpy(), drift)
