"""The work that a serving program has the region-sparse DiT step do, as timed cases.

Kinds (every one through the binding's public entry points):

  step        SparseStep.step: score, select, gather, embed, adaLN of every block, the blocks, final
              layer, latent update.  The sampler keeps x_n (the next step's x_prev), so the step
              runs in place on a copy of it.
  block       fd_embed and one fd_block_forward on the active rows of a batch: the DiT block that a
              step repeats 24 or 30 times, with the modulation from fd_adaln (as in a step) or its own.
  gate        the step without the network: fd_region_score, fd_select, fd_gather, fd_scatter_update.
  importance  fd_region_importance after a block (the Patch Gate's own signal, once per step).
  partition   fd_partition of the requests' saliency maps (once per request).
  head        fd_adaln of all blocks and fd_final: the step's conditioning and its last layer.

`requests` is text: comma-separated COUNT*DIMS (1, 2 or 3 axes), or COUNT*LO~HI for sequences of odd
lengths between LO and HI.  `region` is the region size per axis (clipped at the grid's edge), `frac`
the share of each request's regions that is active.  Model sizes are the package's workloads' (tiny,
audio, image, video) and one generic small model.  Weights and latents follow the workloads' recipe:
weights N(0, 0.02) in bf16, latents N(0, 1), hot regions moving by U[1, 2] and cold ones by
U[0.05, 0.45], the threshold between the two.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_12121_amd import flashdiff as fdl

# C, D, H, dh, F
MODELS = {"tiny": (16, 64, 4, 16, 256), "small": (32, 384, 6, 64, 1536), "audio": (64, 1024, 16, 64, 4096),
          "image": (64, 1536, 24, 64, 6144), "video": (64, 1536, 12, 128, 6144)}
DT = -0.02


def listed():
    return [
        # the smallest call: a whole step of the tiny model, where launches and host work are all there is;
        # skipped regions move with their cached drift
        dict(name="step_tiny", kind="step", model="tiny", blocks=1, requests="1*16x16", region="4x4", frac=0.5, drift=True),
        # a whole step of one 1024^2 image request: what one user waits for, 50 times an image
        dict(name="step_image", kind="step", model="image", blocks=24, requests="1*64x64", region="8x8", frac=0.41, drift=False),
        # its block alone
        dict(name="block_image", kind="block", model="image", requests="1*64x64", region="8x8", frac=0.41, own_adaln=False),
        # the largest: the block of one video request, 30% of 32760 tokens active, head dim 128
        dict(name="block_video", kind="block", model="video", requests="1*21x30x52", region="3x6x13", frac=0.3, own_adaln=False),
        # a short sequence on a narrower model
        dict(name="block_audio", kind="block", model="audio", requests="1*2048", region="32", frac=0.5, own_adaln=False),
        # a serving batch of images of three sizes
        dict(name="block_packed", kind="block", model="image", requests="2*32x32,3*48x48,3*64x64", region="8x8", frac=0.45,
             own_adaln=False),
        # the dense warm-up of many short requests of odd lengths (every row active, as a prefill),
        # the block forming its own modulation
        dict(name="block_warmup", kind="block", model="audio", requests="48*65~511", region="32", frac=1.0, own_adaln=True),
        # the gate side of a video step, cached-drift update
        dict(name="gate_video", kind="gate", channels=64, requests="1*21x30x52", region="3x6x13", frac=0.3, drift=True),
        # the gate side of a full batch: 64 image requests, skipped regions frozen
        dict(name="gate_batch", kind="gate", channels=64, requests="64*64x64", region="8x8", frac=0.41, drift=False),
        # the gate signal of a video step with the importance gate
        dict(name="importance_video", kind="importance", model="video", requests="1*21x30x52", region="3x6x13", frac=0.3),
        # the partitioner on the saliency maps of a batch of images
        dict(name="partition_packed", kind="partition", requests="2*32x32,3*48x48,3*64x64", region="8x8", levels=4096),
        # the conditioning of all 24 blocks of the image model and its final layer
        dict(name="head_image", kind="head", model="image", blocks=24, requests="1*64x64", region="8x8", frac=0.41),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_requests(rng, total):
    """About `total` tokens in one or several requests: (requests, region)."""
    n_req = min(_log(rng, 1, 48), max(1, total // 64))
    per = max(64, total // n_req)
    if rng.random() < 0.5:   # images
        y = max(5, int(round(math.sqrt(per) * rng.uniform(0.7, 1.4))))
        x = max(5, per // y)
        return "%d*%dx%d" % (n_req, y, x), "%dx%d" % ((8, 8) if per >= 256 else (4, 4))
    if n_req == 1:
        return "1*%d" % (per + rng.randint(0, 31)), "%d" % rng.choice((32, 48, 64))
    return "%d*%d~%d" % (n_req, max(33, per // 2), per + per // 2), "%d" % rng.choice((32, 48, 64))


def draw(rng):
    kind = rng.choice(("block", "block", "block", "block", "step", "gate", "gate", "importance", "partition", "head"))
    if kind == "block" or kind == "importance":
        model = rng.choice(("small", "audio", "image", "video"))
        total = _log(rng, 256, 32760)
        requests, region = _draw_requests(rng, total)
        frac = round(rng.uniform(0.05, 0.3) if total > 8192 else rng.uniform(0.05, 1.0), 3)
        c = dict(kind=kind, model=model, requests=requests, region=region, frac=frac)
        if kind == "block":
            c["own_adaln"] = rng.random() < 0.3
        return c
    if kind == "step":
        model = rng.choice(("tiny", "small", "audio"))
        requests, region = _draw_requests(rng, _log(rng, 256, 4096))
        return dict(kind=kind, model=model, blocks=rng.randint(1, 6), requests=requests, region=region,
                    frac=round(rng.uniform(0.1, 0.9), 3), drift=rng.random() < 0.5)
    if kind == "gate":
        requests, region = _draw_requests(rng, _log(rng, 256, 131072))
        return dict(kind=kind, channels=rng.choice((16, 64, 64, 128)), requests=requests, region=region,
                    frac=round(rng.uniform(0.1, 0.9), 3), drift=rng.random() < 0.5)
    if kind == "partition":
        requests, region = _draw_requests(rng, _log(rng, 256, 32760))
        return dict(kind=kind, requests=requests, region=region, levels=rng.choice((256, 4096, 65536)))
    requests, region = _draw_requests(rng, _log(rng, 256, 8192))
    return dict(kind="head", model=rng.choice(("small", "audio", "image")), blocks=rng.randint(1, 24), requests=requests,
                region=region, frac=round(rng.uniform(0.1, 1.0), 3))


# ------------------------------------------------------------------ layout

def _layout(case):
    """token -> region (global), request token offsets, request region offsets."""
    region = [int(v) for v in case["region"].split("x")]
    maps, tok, reg = [], [0], [0]
    for part in case["requests"].split(","):
        count, dims = part.split("*")
        if "~" in dims:
            lo, hi = (int(v) for v in dims.split("~"))
            shapes = [[int(v)] for v in np.random.default_rng([int(count), lo, hi]).integers(lo, hi + 1, int(count))]
        else:
            shapes = [[int(v) for v in dims.split("x")]] * int(count)
        for shape in shapes:
            grid = [-(-n // r) for n, r in zip(shape, region)]
            at = np.indices(shape).reshape(len(shape), -1)
            rid = np.zeros(at.shape[1], np.int64)
            for axis, (r, g) in enumerate(zip(region, grid)):
                rid = rid * g + at[axis] // r
            maps.append(rid + reg[-1])
            tok.append(tok[-1] + at.shape[1])
            reg.append(reg[-1] + int(np.prod(grid)))
    return np.concatenate(maps).astype(np.int32), np.asarray(tok, np.int32), np.asarray(reg, np.int32)


def _active(case, seed, reg_off):
    """The regions that move: `frac` of every request's, at least one."""
    rng = np.random.default_rng([seed, 7])
    act = np.zeros(reg_off[-1], bool)
    for lo, hi in zip(reg_off[:-1], reg_off[1:]):
        act[lo + rng.permutation(hi - lo)[:max(1, int(round(case["frac"] * (hi - lo))))]] = True
    return act


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, *shape, std=1.0, dtype=torch.float32):
    return (torch.randn(shape, generator=g, device="cuda") * std).to(dtype)


def _inputs(case, seed):
    """Everything that comes from the seed, as plain tensors and arrays."""
    t = {}
    tr, tok_off, reg_off = _layout(case)
    t.update(token_region=tr, tok_off=tok_off, reg_off=reg_off)
    N, B, R = len(tr), len(tok_off) - 1, int(reg_off[-1])
    kind = case["kind"]
    if kind == "partition":
        # a few objects on a weak background, quantised (concentrated, as cross-attention of salient words)
        rng, maps = np.random.default_rng([seed, 3]), []
        for b in range(B):
            n = int(tok_off[b + 1] - tok_off[b])
            side = max(1, int(round(math.sqrt(n))))
            at = np.stack([np.arange(n) // side, np.arange(n) % side]) / side
            field = rng.uniform(0.0, 0.05, n)
            for _ in range(int(rng.integers(3, 7))):
                z = (at - rng.uniform(0.0, 1.0, (2, 1))) / rng.uniform(0.05, 0.25, (2, 1))
                field += rng.uniform(0.3, 1.0) * np.exp(-0.5 * (z ** 2).sum(axis=0))
            maps.append(np.floor(field / field.max() * (case["levels"] - 1)).astype(np.uint16))
        t["saliency"] = torch.from_numpy(np.concatenate(maps).view(np.int16)).cuda()
        return t
    g = _generator(seed)
    act = _active(case, seed, reg_off)
    tok = np.nonzero(act[tr])[0]
    t.update(act=act, tok=tok, M=len(tok))
    t["cu_q"] = np.searchsorted(tok, tok_off).astype(np.int32)
    if kind in ("gate", "step"):
        C = case["channels"] if kind == "gate" else MODELS[case["model"]][0]
        rng = np.random.default_rng([seed, 11])
        amp = np.where(act, rng.uniform(1.0, 2.0, R), rng.uniform(0.05, 0.45, R))
        eps = np.zeros(B)
        for b in range(B):
            e, a = amp[reg_off[b]:reg_off[b + 1]] ** 2, act[reg_off[b]:reg_off[b + 1]]
            eps[b] = 0.0 if a.all() else 0.5 * (e[~a].max() + e[a].min()) / e.sum()
        t["x_prev"] = _normal(g, N, C)
        t["x"] = t["x_prev"] + torch.from_numpy(amp[tr].astype(np.float32)).cuda()[:, None] * _normal(g, N, C)
        t["eps"] = torch.from_numpy(eps).cuda()
        t["dt"] = torch.full((B,), DT, dtype=torch.float32, device="cuda")
        t["vcache"] = _normal(g, N, C)
        t["C"] = C
    if kind == "gate":
        t["v"] = _normal(g, N, C)
        return t
    C, D, H, dh, F = MODELS[case["model"]]
    L = case.get("blocks", 1)
    bf = torch.bfloat16
    t["cond"] = _normal(g, B, D)
    if kind != "head":
        shapes = dict(w_qkv=(3 * D, D), b_qkv=(3 * D,), w_o=(D, D), b_o=(D,), w_1=(F, D), b_1=(F,), w_2=(D, F), b_2=(D,),
                      w_ada=(6 * D, D), b_ada=(6 * D,))
        t["params"] = {k: _normal(g, L, *s, std=0.02, dtype=bf if k[0] == "w" else torch.float32) for k, s in shapes.items()}
        t["params"].update(w_e=_normal(g, D, C, std=0.02, dtype=bf), b_e=_normal(g, D, std=0.02),
                           pos=_normal(g, N, D, std=0.02))
        t["k_cache"], t["v_cache"] = _normal(g, L, N, D, dtype=bf), _normal(g, L, N, D, dtype=bf)
    else:
        t["params"] = dict(w_ada=_normal(g, L, 6 * D, D, std=0.02, dtype=bf), b_ada=_normal(g, L, 6 * D, std=0.02))
        t["h"] = _normal(g, N, D)
    if kind in ("head", "step"):
        t["params"].update(w_adaf=_normal(g, 2 * D, D, std=0.02, dtype=bf), b_adaf=_normal(g, 2 * D, std=0.02),
                           w_out=_normal(g, C, D, std=0.02, dtype=bf), b_out=_normal(g, C, std=0.02))
    if kind in ("block", "importance"):
        t["xa"] = _normal(g, N, C, dtype=bf)   # rows < M are the gathered latent rows
    return t


# ------------------------------------------------------------------ state and pass

class _State:
    pass


def _buffers(s, t):
    """idx, cu_q and m as fd_select leaves them, on the device."""
    N = len(t["token_region"])
    s.idx = torch.zeros(N, dtype=torch.int32, device="cuda")
    s.idx[:t["M"]] = torch.from_numpy(t["tok"].astype(np.int32)).cuda()
    s.cu_q = torch.from_numpy(t["cu_q"]).cuda()
    s.m = torch.tensor([t["M"]], dtype=torch.int32, device="cuda")
    s.active = torch.from_numpy(t["act"].astype(np.uint8)).cuda()


def prepare(case, seed):
    t = _inputs(case, seed)
    s = _State()
    s.t, s.case = t, case
    N, B, R = len(t["token_region"]), len(t["tok_off"]) - 1, int(t["reg_off"][-1])
    kind = case["kind"]
    if kind == "partition":
        s.region = torch.zeros(N, dtype=torch.int32, device="cuda")
        s.ws = torch.empty(max(fdl.fd_partition_ws_size(N, B), 256), dtype=torch.uint8, device="cuda")
        return s
    s.plan = fdl.make_plan(t["token_region"], t["tok_off"], R)
    s.ones = torch.ones(R, dtype=torch.uint8, device="cuda")
    if kind == "gate":
        C = t["C"]
        s.x = t["x"].clone()
        s.vcache = t["vcache"].clone()
        s.score, s.s_tilde = (torch.zeros(R, dtype=torch.float64, device="cuda") for _ in range(2))
        s.skip_run = torch.zeros(R, dtype=torch.int32, device="cuda")
        s.active = torch.ones(R, dtype=torch.uint8, device="cuda")
        s.idx = torch.zeros(N, dtype=torch.int32, device="cuda")
        s.cu_q = torch.zeros(B + 1, dtype=torch.int32, device="cuda")
        s.m = torch.zeros(1, dtype=torch.int32, device="cuda")
        s.xa = torch.zeros((N, C), dtype=torch.bfloat16, device="cuda")
        s.ws = torch.empty(max(fdl.fd_region_score_ws_size(s.plan, C), 256), dtype=torch.uint8, device="cuda")
        return s
    C, D, H, dh, F = MODELS[case["model"]]
    s.d = fdl.dims(C, D, H, dh, F)
    L = case.get("blocks", 1)
    if kind == "step":
        s.step = fdl.SparseStep(s.plan, s.d, t["params"], L, k_cache=t["k_cache"].clone(), v_cache=t["v_cache"].clone())
        s.step.vcache.copy_(t["vcache"])
        s.x = t["x"].clone()
        return s
    _buffers(s, t)
    s.ws = torch.empty(fdl.fd_block_ws_size(s.plan, s.d), dtype=torch.uint8, device="cuda")
    if kind == "head":
        s.mod = torch.zeros((L, B, 6 * D), dtype=torch.float32, device="cuda")
        s.v = torch.zeros((N, C), dtype=torch.float32, device="cuda")
        s.w = fdl.final_weights(t["params"])
        return s
    s.h = torch.zeros((N, D), dtype=torch.float32, device="cuda")
    s.k, s.v = t["k_cache"][0].clone(), t["v_cache"][0].clone()
    s.mod = None
    if not case.get("own_adaln"):
        s.mod = torch.zeros((B, 6 * D), dtype=torch.float32, device="cuda")
        fdl.fd_adaln(s.d, 1, 6 * D, B, t["params"]["w_ada"], t["params"]["b_ada"], t["cond"], s.mod)
    s.w = fdl.block_weights(t["params"], 0, s.mod)
    if kind == "importance":
        _run_block(s)
        s.r_bar, s.delta, s.importance = (torch.zeros(R, dtype=torch.float64, device="cuda") for _ in range(3))
        s.ws_imp = torch.empty(max(fdl.fd_importance_ws_size(s.plan, s.d), 256), dtype=torch.uint8, device="cuda")
    return s


def _run_block(s):
    t, p = s.t, s.t["params"]
    fdl.fd_embed(s.plan, s.d, t["xa"], p["w_e"], p["b_e"], p["pos"], s.idx, s.m, s.h)
    fdl.fd_block_forward(s.plan, s.d, s.w, t["cond"], s.h, s.idx, s.cu_q, s.m, s.k, s.v, s.ws)


def run(s):
    case, t = s.case, s.t
    kind = case["kind"]
    if kind == "block":
        _run_block(s)
        return {"h": s.h, "k_cache": s.k, "v_cache": s.v}
    if kind == "step":
        st = s.step
        s.x.copy_(t["x"])
        st.step(s.x, t["x_prev"], t["eps"], t["dt"], t["cond"], stateless=True,
                skip_mode=fdl.FD_SKIP_REUSE_DRIFT if case["drift"] else fdl.FD_SKIP_FREEZE)
        return {"x": s.x, "v": st.v, "vcache": st.vcache, "h": st.h, "k_cache": st.k_cache, "v_cache": st.v_cache,
                "score": st.score, "active": st.active, "idx": st.idx, "cu_q": st.cu_q, "m": st.m}
    if kind == "gate":
        C = t["C"]
        if case["drift"]:   # every region moves: on a copy, as in a step, so that the same regions stay hot
            s.x.copy_(t["x"])
        fdl.fd_region_score(s.plan, C, s.x, t["x_prev"], s.score, s.ws)
        fdl.fd_select(s.plan, s.score, t["eps"], 0.0, 0, s.s_tilde, s.skip_run, s.ones, s.active, s.idx, s.cu_q, s.m)
        fdl.fd_gather(s.plan, C, s.x, s.idx, s.m, s.xa)
        fdl.fd_scatter_update(s.plan, C, s.x, t["v"], s.idx, s.m, t["dt"], s.vcache, s.active,
                              fdl.FD_SKIP_REUSE_DRIFT if case["drift"] else fdl.FD_SKIP_FREEZE)
        return {"score": s.score, "s_tilde": s.s_tilde, "skip_run": s.skip_run, "active": s.active, "idx": s.idx,
                "cu_q": s.cu_q, "m": s.m, "xa": s.xa, "x": s.x, "vcache": s.vcache}
    if kind == "importance":
        fdl.fd_region_importance(s.plan, s.d, s.ws, s.k, s.idx, s.m, s.active, s.r_bar, s.delta, s.importance, s.ws_imp)
        return {"importance": s.importance, "r_bar": s.r_bar, "delta": s.delta}
    if kind == "partition":
        fdl.fd_partition(t["tok_off"], t["reg_off"], t["saliency"], s.region, s.ws)
        return {"region": s.region}
    C, D, H, dh, F = MODELS[case["model"]]
    fdl.fd_adaln(s.d, case["blocks"], 6 * D, s.plan.n_requests, t["params"]["w_ada"], t["params"]["b_ada"], t["cond"], s.mod)
    fdl.fd_final(s.plan, s.d, s.w, t["cond"], t["h"], s.cu_q, s.m, s.v, s.ws)
    return {"mod": s.mod, "v": s.v}


# ------------------------------------------------------------------ work and tolerance

def work(case):
    tr, tok_off, reg_off = _layout(case)
    N, B, R = len(tr), len(tok_off) - 1, int(reg_off[-1])
    kind = case["kind"]
    if kind == "partition":
        return {"bytes": 6 * N, "flops": 0}
    n_b = np.diff(tok_off).astype(np.float64)
    m_b = case["frac"] * n_b
    M = float(m_b.sum())
    if kind == "gate" or kind == "step":
        C = case["channels"] if kind == "gate" else MODELS[case["model"]][0]
        # score: both latents; gather; update of the active rows (and of the skipped ones with their drift)
        gate = 8 * N * C + 16 * R + 4 * N + M * (6 * C + 4) + M * 16 * C + (12 * (N - M) * C if case["drift"] else 0)
        if kind == "gate":
            return {"bytes": gate, "flops": 3 * N * C}
    C, D, H, dh, F = MODELS[case["model"]]
    L = case.get("blocks", 1)
    block_fl = 2 * M * (4 * D * D + 2 * D * F) + 4 * D * float((m_b * n_b).sum())
    # weights, hidden rows in and out, K/V of every token read, fresh K/V rows written
    block_by = 2 * (4 * D * D + 2 * D * F) + 8 * M * D + 4 * N * D + 4 * M * D
    ada_by, ada_fl = 12 * D * D + 24 * B * D, 12 * B * D * D
    embed_by, embed_fl = M * (2 * C + 8 * D) + 2 * D * C, 2 * M * C * D
    final_by, final_fl = 4 * D * D + M * (4 * D + 4 * C), 4 * B * D * D + 2 * M * C * D
    if kind == "block":
        own = case["own_adaln"]
        return {"bytes": block_by + embed_by + own * ada_by, "flops": block_fl + embed_fl + own * ada_fl}
    if kind == "importance":
        n_r = np.bincount(tr).astype(np.float64)
        return {"bytes": 4 * M * D + 4 * M * H + 24 * R, "flops": 2 * D * case["frac"] * float((n_r ** 2).sum())}
    if kind == "head":
        return {"bytes": L * ada_by + final_by, "flops": L * ada_fl + final_fl}
    return {"bytes": gate + embed_by + L * (block_by + ada_by) + final_by,
            "flops": embed_fl + L * (block_fl + ada_fl) + final_fl}


def tolerance(case):
    kind = case["kind"]
    if kind == "partition":
        return "exact"
    if kind == "gate":   # scores in 64 bits, everything else one rounding of given values
        return {"rel": 1e-6, "max": 1e-6}
    # about four times the error against 64 bits (importance 5e-5, its sums are over thousands of
    # roundings; a head's velocity 1.7e-3, a block 2.5e-3, 24 blocks 4.3e-3)
    if kind == "importance":
        return {"rel": 3e-4}
    if kind == "head":
        return {"rel": 7e-3}
    return {"rel": 2e-2 if kind == "step" else 1e-2}


# ------------------------------------------------------------------ the same in 64 bits

def _f64(v):
    return v.to(torch.float64)


def _norm64(h):
    z = h - h.mean(dim=-1, keepdim=True)
    return z / torch.sqrt((z * z).mean(dim=-1, keepdim=True) + 1e-6)


def _adaln64(cond, w, b):
    c = _f64(cond)
    return (c * torch.sigmoid(c)) @ _f64(w).T + _f64(b)


def _rows(t):
    """Token and request of every active row, on the device."""
    req = np.repeat(np.arange(len(t["cu_q"]) - 1), np.diff(t["cu_q"]))
    return torch.from_numpy(t["tok"]).cuda(), torch.from_numpy(req).cuda()


def _attend64(t, H, dh, q, k, v, per_head=None):
    """softmax(q k^T / sqrt(dh)) v of the active rows over their requests' tokens."""
    o = torch.zeros_like(q)
    for b in range(len(t["cu_q"]) - 1):
        q0, q1 = int(t["cu_q"][b]), int(t["cu_q"][b + 1])
        k0, k1 = int(t["tok_off"][b]), int(t["tok_off"][b + 1])
        if q1 == q0:
            continue
        for h in range(H):
            c = slice(h * dh, (h + 1) * dh)
            p = torch.softmax(q[q0:q1, c] @ k[k0:k1, c].T.contiguous() / math.sqrt(dh), dim=-1)
            o[q0:q1, c] = p @ v[k0:k1, c].contiguous()
            if per_head is not None:
                per_head(b, p)
    return o


def _block64(t, case, l, h, k, v, per_head=None):
    """One block on the active rows h; k, v (of block l, all tokens) get the fresh rows."""
    C, D, H, dh, F = MODELS[case["model"]]
    p = {n: _f64(w[l]) for n, w in t["params"].items() if n in
         ("w_qkv", "b_qkv", "w_o", "b_o", "w_1", "b_1", "w_2", "b_2")}
    tok, req = _rows(t)
    mod = _adaln64(t["cond"], t["params"]["w_ada"][l], t["params"]["b_ada"][l])
    shift1, scale1, gate1, shift2, scale2, gate2 = (mod[:, i * D:(i + 1) * D][req] for i in range(6))
    a = _norm64(h) * (1 + scale1) + shift1
    q, kn, vn = (a @ p["w_qkv"].T + p["b_qkv"]).split(D, dim=1)
    k[tok], v[tok] = kn, vn
    o = _attend64(t, H, dh, q, k, v, per_head)
    h = h + gate1 * (o @ p["w_o"].T + p["b_o"])
    a = _norm64(h) * (1 + scale2) + shift2
    u = torch.nn.functional.gelu(a @ p["w_1"].T + p["b_1"], approximate="tanh")
    return h + gate2 * (u @ p["w_2"].T + p["b_2"])


def _embed64(t, xa):
    tok, _ = _rows(t)
    p = t["params"]
    return xa @ _f64(p["w_e"]).T + _f64(p["b_e"]) + _f64(p["pos"])[tok]


def _final64(t, h):
    D = h.shape[1]
    _, req = _rows(t)
    p = t["params"]
    mod = _adaln64(t["cond"], p["w_adaf"], p["b_adaf"])
    a = _norm64(h) * (1 + mod[:, D:][req]) + mod[:, :D][req]
    return a @ _f64(p["w_out"]).T + _f64(p["b_out"])


def _all_rows(t, v):
    """The first M of N rows, zeros behind them."""
    out = torch.zeros((len(t["token_region"]), v.shape[1]), dtype=torch.float64, device="cuda")
    out[:t["M"]] = v
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "partition":
        return None
    t = _inputs(case, seed)
    N, R, M = len(t["token_region"]), int(t["reg_off"][-1]), t["M"]
    if kind in ("gate", "step"):
        tok, _ = _rows(t)
        tr = torch.from_numpy(t["token_region"].astype(np.int64)).cuda()
        x = _f64(t["x"])
        size = torch.bincount(tr, minlength=R).to(torch.float64) * t["C"]
        d = _f64(t["x"] - t["x_prev"])   # the method's difference is formed in fp32
        score = torch.zeros(R, dtype=torch.float64, device="cuda").index_add_(0, tr, (d * d).sum(dim=1)) / size
        vcache = _f64(t["vcache"])
        dt = float(np.float32(DT))

        def update(v):
            moved = vcache.clone()
            moved[tok] = v
            go = torch.full((N, 1), 1.0 if case["drift"] else 0.0, dtype=torch.float64, device="cuda")
            go[tok] = 1.0
            return x + dt * go * moved, moved
    if kind == "gate":
        x_new, moved = update(_f64(t["v"][:M]))
        return {"score": score, "s_tilde": score.clone(), "xa": _all_rows(t, x[tok]), "x": x_new, "vcache": moved}
    if kind == "head":
        D = t["h"].shape[1]
        mod = torch.stack([_adaln64(t["cond"], w, b) for w, b in zip(t["params"]["w_ada"], t["params"]["b_ada"])])
        return {"mod": mod, "v": _all_rows(t, _final64(t, _f64(t["h"][:M])))}
    if kind == "step":
        h, ks, vs = _embed64(t, x[tok]), [], []
        for l in range(case["blocks"]):
            k, v = _f64(t["k_cache"][l]), _f64(t["v_cache"][l])
            h = _block64(t, case, l, h, k, v)
            ks.append(k)
            vs.append(v)
        v = _final64(t, h)
        x_new, moved = update(v)
        return {"x": x_new, "v": _all_rows(t, v), "vcache": moved, "h": _all_rows(t, h), "k_cache": torch.stack(ks),
                "v_cache": torch.stack(vs), "score": score}
    k, v = _f64(t["k_cache"][0]), _f64(t["v_cache"][0])
    h = _embed64(t, _f64(t["xa"][:M]))
    if kind == "block":
        h = _block64(t, case, 0, h, k, v)
        return {"h": _all_rows(t, h), "k_cache": k, "v_cache": v}
    H = MODELS[case["model"]][2]
    sums = torch.zeros(R, dtype=torch.float64, device="cuda")
    tr = torch.from_numpy(t["token_region"].astype(np.int64)).cuda()
    row_reg = tr[torch.from_numpy(t["tok"]).cuda()]

    def per_head(b, p):   # the in-region sum of the attention matrix of one request and head
        q0, q1, k0, k1 = (int(t[n][b + i]) for n in ("cu_q", "tok_off") for i in (0, 1))
        r0, n_r = int(t["reg_off"][b]), int(t["reg_off"][b + 1] - t["reg_off"][b])
        by_region = torch.zeros((q1 - q0, n_r), dtype=torch.float64, device="cuda").index_add_(1, tr[k0:k1] - r0, p)
        mine = by_region.gather(1, (row_reg[q0:q1] - r0)[:, None])[:, 0]
        sums.index_add_(0, row_reg[q0:q1], mine)

    _block64(t, case, 0, h, k, v, per_head)
    n = torch.bincount(tr, minlength=R).to(torch.float64)
    imp = sums / (H * n * n)
    act = torch.from_numpy(t["act"]).cuda()
    zero = torch.zeros_like(imp)
    return {"importance": torch.where(act, imp, torch.full_like(imp, math.nan)), "r_bar": torch.where(act, imp, zero),
            "delta": torch.where(act, imp, zero)}
