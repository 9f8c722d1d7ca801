"""Blocks whose operands are larger than the 2 GiB that a 32-bit buffer offset reaches: the MLP's
activations (both GEMM kernels read them) and the K/V caches.  The rows of the last request, the ones
past that line, against the block in float64."""
import math

import numpy as np
import pytest
import torch

from paper_2607_12121_amd import flashdiff as fdl
from tests import gpu_harness as gh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    fdl.lib()
    yield
    torch.cuda.empty_cache()


def _block64(h, p, mod, H, k, v):
    """One block of one request: all of its rows h active, K/V rows fresh."""
    D = h.shape[1]
    norm = lambda x: torch.nn.functional.layer_norm(x, (D,), eps=1e-6)
    w = {n: t[0].double() for n, t in p.items()}
    sh1, sc1, g1, sh2, sc2, g2 = mod.double().split(D)
    q, kf, vf = ((norm(h) * (1 + sc1) + sh1) @ w["w_qkv"].T.contiguous() + w["b_qkv"]).split(D, dim=1)
    k, v = torch.cat([k.double(), kf]), torch.cat([v.double(), vf])
    dh, o = D // H, torch.empty_like(q)
    for i in range(H):
        c = slice(i * dh, (i + 1) * dh)
        o[:, c] = torch.softmax(q[:, c] @ k[:, c].T.contiguous() / math.sqrt(dh), dim=-1) @ v[:, c].contiguous()
    h = h + g1 * (o @ w["w_o"].T.contiguous() + w["b_o"])
    a = norm(h) * (1 + sc2) + sh2
    u = torch.nn.functional.gelu(a @ w["w_1"].T.contiguous() + w["b_1"], approximate="tanh")
    return h + g2 * (u @ w["w_2"].T.contiguous() + w["b_2"])


@pytest.mark.parametrize("D,H,dh,F,sizes,active,what", [
    (64, 1, 64, 32832, [1000] * 33, "all", "activations"),        # narrow down-projection
    (1024, 16, 64, 16384, [1025] * 64, "all", "activations"),     # the 512-thread kernel
    (1024, 16, 64, 64, [1 << 20, 1000], "last", "caches"),
    (1024, 8, 128, 64, [1 << 20, 1000], "last", "caches"),
])
def test_block_past_2_gib(D, H, dh, F, sizes, active, what):
    N, B, n = sum(sizes), len(sizes), sizes[-1]
    M = N if active == "all" else n
    assert (M * F if what == "activations" else N * D) * 2 > 1 << 31
    gh.say(f"block past 2 GiB of {what}: D={D} dh={dh} F={F} tokens={N}")
    g = torch.Generator(device="cuda")
    g.manual_seed(D + F + dh)
    draw = lambda *s, std=1.0, dtype=torch.float32: (torch.randn(s, generator=g, device="cuda", dtype=dtype) * std)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    plan = fdl.make_plan(np.repeat(np.arange(B), sizes).astype(np.int32), off, B)
    d = fdl.dims(64, D, H, dh, F)
    shapes = dict(w_qkv=(3 * D, D), b_qkv=(3 * D,), w_o=(D, D), b_o=(D,), w_1=(F, D), b_1=(F,), w_2=(D, F), b_2=(D,),
                  w_ada=(8,), b_ada=(8,))
    p = {k: draw(1, *s, std=2.0 / math.sqrt(s[-1]) if k[0] == "w" else 0.02,
                 dtype=torch.bfloat16 if k[0] == "w" else torch.float32) for k, s in shapes.items()}
    mod = draw(B, 6 * D, std=0.5)
    kc, vc = (draw(N, D, dtype=torch.bfloat16) for _ in range(2))
    h = draw(N, D)
    idx = torch.arange(N - M, N, dtype=torch.int32, device="cuda")
    idx = torch.cat([idx, torch.zeros(N - M, dtype=torch.int32, device="cuda")])
    cu = torch.from_numpy(off if active == "all" else np.array([0] * B + [n], np.int32)).cuda()
    m = torch.tensor([M], dtype=torch.int32, device="cuda")
    ws = torch.empty(fdl.fd_block_ws_size(plan, d), dtype=torch.uint8, device="cuda")
    rows = slice(M - n, M)
    before = h[rows].double()
    want = _block64(before, p, mod[-1], H, kc[:0], vc[:0])
    fdl.fd_block_forward(plan, d, fdl.block_weights(p, 0, mod), None, h, idx, cu, m, kc, vc, ws)
    got = h[rows].double()
    scale = (want - before).abs().max()
    assert ((got - want).abs().max() / scale).item() <= gh.TOL
    # the rows past the line by themselves
    assert ((got[-32:] - want[-32:]).norm() / (want[-32:] - before[-32:]).norm()).item() <= 1e-2
