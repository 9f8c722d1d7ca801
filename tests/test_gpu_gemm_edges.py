"""The GEMM variants at the sizes where they change: the embedding with channel counts
that are and are not a multiple of 64, at the edges of its 128-row tiles; the down-projection where its split count changes; every
tile shape of the long batches' kernel, its pairs of tiles with work in both groups, and the row
capacity from which it runs."""
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


@pytest.mark.parametrize("C", [16, 48, 64, 80, 144, 256])
@pytest.mark.parametrize("M,N,D", [(1, 1, 64), (127, 127, 192), (128, 300, 64), (129, 129, 128), (0, 40, 64), (513, 700, 320)])
def test_embed_edges(C, M, N, D):
    """M active rows of N tokens: h = xa w^T + b + pos[idx], rows past M untouched.  The products
    of bf16 values are exact in fp32, so only the order of C + 2 fp32 additions differs from the
    float64 result: each row's error is at most (C + 2) 2^-24 of the sum of magnitudes."""
    gh.say(f"embed C={C} M={M} N={N} D={D}")
    rng = np.random.default_rng([C, M, N, D])
    dims = fdl.dims(C, D, D // 64, 64, 64)
    plan = fdl.make_plan(np.zeros(N, np.int32), np.array([0, N], np.int32), 1)
    idx = np.sort(rng.permutation(N)[:M]).astype(np.int32)
    xa = torch.from_numpy(rng.standard_normal((N, C)).astype(np.float32)).to(torch.bfloat16)
    w = torch.from_numpy(rng.standard_normal((D, C)).astype(np.float32)).to(torch.bfloat16)
    b = torch.from_numpy(rng.standard_normal(D).astype(np.float32))
    pos = torch.from_numpy(rng.standard_normal((N, D)).astype(np.float32))
    h = torch.full((N, D), -7.0, device="cuda")
    d_idx = torch.zeros(N, dtype=torch.int32, device="cuda")
    d_idx[:M] = torch.from_numpy(idx).cuda()
    fdl.fd_embed(plan, dims, xa.cuda(), w.cuda(), b.cuda(), pos.cuda(), d_idx,
                 torch.tensor([M], dtype=torch.int32, device="cuda"), h)
    got = h.cpu().double().numpy()
    x64, w64, p64 = xa.double().numpy()[:M], w.double().numpy(), pos.double().numpy()[idx]
    want = x64 @ w64.T + b.double().numpy() + p64
    bound = (C + 2) * 2.0 ** -24 * (np.abs(x64) @ np.abs(w64).T + np.abs(b.double().numpy()) + np.abs(p64))
    assert np.all(np.abs(got[:M] - want) <= bound)
    assert np.all(got[M:] == -7.0)


@pytest.mark.parametrize("C", [48, 64])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_embed_unaligned_tables(C, shift):
    """A position table and an output that start `shift` floats past a 16-byte line: the same bits
    as aligned ones."""
    M, N, D = 129, 200, 192
    gh.say(f"embed unaligned C={C} shift={shift}")
    rng = np.random.default_rng([C, shift])
    dims = fdl.dims(C, D, D // 64, 64, 64)
    plan = fdl.make_plan(np.zeros(N, np.int32), np.array([0, N], np.int32), 1)
    idx = torch.zeros(N, dtype=torch.int32, device="cuda")
    idx[:M] = torch.from_numpy(np.sort(rng.permutation(N)[:M]).astype(np.int32)).cuda()
    xa, w = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).to(torch.bfloat16).cuda() for s in ((N, C), (D, C)))
    b, pos = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).cuda() for s in ((D,), (N, D)))
    m = torch.tensor([M], dtype=torch.int32, device="cuda")
    out = []
    for s in (0, shift):
        p, h = (torch.zeros(N * D + s, device="cuda")[s:].view(N, D) for _ in range(2))
        assert p.data_ptr() % 16 == 4 * s and h.data_ptr() % 16 == 4 * s
        p.copy_(pos)
        fdl.fd_embed(plan, dims, xa, w, b, p, idx, m, h)
        out.append(h[:M].clone())
    assert torch.equal(*out)


@pytest.mark.parametrize("F", [1984, 2048, 3072])
@pytest.mark.parametrize("tokens,frac", [((40,), 1.0), ((129, 300), 0.5)])
def test_block_split_edges(F, tokens, frac):
    """A block whose down-projection has 31 (no split), 32 (two splits) and 48 (three) K-steps."""
    w = small_workload("audio", requests=tuple(wl.RequestShape("seq", (n,), (16,)) for n in tokens), activity="frac",
                       activity_args=(frac, 1.0), L=1, D=128, H=2, dh=64, F=F)
    case = gh.make_case("audio", workload=w)
    gh.say(f"split edges F={F} tokens={tokens}")
    g, st = gh.run_gpu(case, case.inp.eps, case.inp.x_cur, case.inp.x_prev)
    o = gh.run_oracle(case, case.inp.eps, case.inp.x_cur, case.inp.x_prev)
    gh.compare_step(case, g, o, case.inp.x_cur, st)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("requests,region,active", [(1, 25, 1), (1, 25, 41), (82, 20, 2), (82, 20, 5)])
def test_large_kernel_shapes(requests, region, active):
    """8200 tokens at hidden 1024 run the 512-thread kernel.  `active` regions per request: 25 rows
    (128x64 tiles, the second group of every workgroup without a unit; the down-projection's 128x128
    tiles split in two), 1025 rows (128x128 with a last tile of one row, 128x64), 3280 (192x256 and
    128x256, ragged last tiles) and 8200 (256x256)."""
    _shapes(requests, region, active, 8200, 1024, 2048)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("active", [10, 20, 29, 58])
def test_large_kernel_pairs(active):
    """Hidden 1088 (columns an odd number of 64s) runs two 128x64 tiles per workgroup: QKV at 1280 rows
    (510 units: the second group of two workgroups has none) and 2560 (1020 units, two each, ends
    unequal), the out- and down-projections at 3712 (493) and 7424 rows (986)."""
    _shapes(1, 128, active, 8320, 1088, 1088)


def _shapes(requests, region, active, tokens, D, F):
    w = small_workload("audio", requests=tuple(wl.RequestShape("seq", (tokens // requests,), (region,)) for _ in range(requests)),
                       activity="count", activity_args=(active,), L=1, D=D, H=D // 64, dh=64, F=F)
    case = gh.make_case("audio", workload=w)
    eps = np.zeros(requests) if (requests, active) == (82, 5) else case.inp.eps
    gh.say(f"large kernel shapes: D={D}, {requests} requests, {active} active regions each")
    g, st = gh.run_gpu(case, eps, case.inp.x_cur, case.inp.x_prev)
    M = requests * active * region
    assert g["M"] == M
    rows = np.unique(np.concatenate([[0, M - 1], np.random.default_rng(3).choice(M, min(M, 126), replace=False)]))
    o = gh.run_oracle(case, eps, case.inp.x_cur, case.inp.x_prev, sample_rows=rows)
    gh.compare_step(case, g, o, case.inp.x_cur, st)


@pytest.mark.parametrize("tokens", [8191, 8192])
@pytest.mark.parametrize("active", [1, 30])
def test_large_kernel_line(tokens, active):
    """One token on either side of the capacity from which the 512-thread kernel runs, few rows
    (the down-projection's split) and more."""
    w = small_workload("audio", requests=(wl.RequestShape("seq", (tokens,), (32,)),), activity="count",
                       activity_args=(active,), L=1, D=1024, H=16, dh=64, F=2048)
    case = gh.make_case("audio", workload=w)
    gh.say(f"large kernel line: {tokens} tokens, {active} active regions")
    g, st = gh.run_gpu(case, case.inp.eps, case.inp.x_cur, case.inp.x_prev)
    M = g["M"]
    rows = np.unique(np.concatenate([[0, M - 1], np.random.default_rng(3).choice(M, min(M, 62), replace=False)]))
    o = gh.run_oracle(case, case.inp.eps, case.inp.x_cur, case.inp.x_prev, sample_rows=rows)
    gh.compare_step(case, g, o, case.inp.x_cur, st)
