"""The calls whose speed is measured: the work that users of this package have it do.

A case is a dict of plain values:

    entry   which public entry point a pass goes through:
              "tiled"  ns_tiled over a list of matrices (the tiled map)
              "gemm"   ns_gemm over a list of matrices (T = 512 tiles, or T = 0
                       for whole matrices)
              "step"   one HiMuon.step (momentum, map, weight update)
    shapes  "HxW,HxW,..." or "N*HxW,..." (N matrices of one shape)
    dtype   storage type of the matrices
    T, K    tile size (0: whole matrices) and Newton-Schulz steps
    data    "lowrank" (a momentum-like matrix: rank 64 with a 1/i spectrum, plus
            noise), "gauss" or "heavy" (0.02 t(3), the heavy-tailed gradients)

Shapes are those of this repository's workloads and tests (one 7B-style layer,
the Qwen3 blocks, the heterogeneous batch, N x Linear(H, H), a 256 x 256 matrix)
or generic.
"""
import math

import numpy as np
import torch
import torch.nn.functional as F

import paper_2606_27216_amd as hm

COEFFS = tuple(float(np.float32(v)) for v in hm.QUINTIC)  # what the library computes with
LR, BETA, DECAY, SCALE = 0.02, 0.95, 0.1, 0.2

LAYER_7B = "4*4096x4096,2*11008x4096,4096x11008"
QWEN_06B = "2048x1024,2*1024x1024,1024x2048,2*3072x1024,1024x3072"
QWEN_17B = "2*2048x2048,2*1024x2048,2*6144x2048,2048x6144"
HETERO = "8*1024x4096,8*4096x1024,8*2048x2048"


def _case(name, entry, shapes, dtype, T, K=5, data="lowrank"):
    return {"name": name, "entry": entry, "shapes": shapes, "dtype": dtype, "T": T, "K": K, "data": data}


def listed():
    return [
        # the smallest call: one small fp32 matrix, 64 tiles in one launch
        _case("f32_256_T32", "tiled", "256x256", "f32", 32, data="gauss"),
        # per-layer calls of a small model's optimizer: one projection at a time
        _case("one_1024_T128", "tiled", "1024x1024", "bf16", 128),
        _case("one_2048x1024_T512", "gemm", "2048x1024", "bf16", 512),
        # a transformer block's optimizer step in one call, the tile size that
        # training ends with
        _case("step_block06_T128", "step", QWEN_06B, "bf16", 128),
        # the optimizer-step study's batch at the tile size that it uses
        _case("step_8x2048_T512", "step", "8*2048x2048", "bf16", 512),
        # the start of training: whole matrices, a block of the 1.7B model
        _case("step_block17_full", "step", QWEN_17B, "bf16", 0),
        # matrices whose sizes are no multiples of anything: vocabulary heads,
        # pruned or odd hidden sizes; rows are then not 16-byte aligned either
        _case("ragged_T128", "tiled", "1000x1003,300x420,33x4096,2*777x3001,1531x2050", "bf16", 128, data="gauss"),
        # the runtime tile-size schedule on the heterogeneous batch
        _case("square4096_T256", "tiled", "4096x4096", "bf16", 256),
        _case("hetero_T64", "tiled", HETERO, "bf16", 64, data="heavy"),
        _case("hetero_f32_T128_K8", "tiled", HETERO, "f32", 128, K=8, data="heavy"),
        _case("hetero_f32_T64", "tiled", HETERO, "f32", 64, data="heavy"),
        # one 7B-style layer, the unit of the large stack
        _case("layer7b_T128", "tiled", LAYER_7B, "bf16", 128),
    ]


def _shapes(case):
    out = []
    for part in case["shapes"].split(","):
        n, _, hw = part.rpartition("*")
        h, w = hw.split("x")
        out += [(int(h), int(w))] * int(n or 1)
    return out


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed kinds: every tile size and both storage
    types on the tiled path, T = 512 and whole matrices on the others; one to
    sixteen matrices of up to three shapes, half of the dimensions multiples of
    64 and half of any size."""
    while True:
        kind = rng.choice(["tiled", "tiled", "tiled", "tiled32", "step", "gemm", "step_gemm"])
        case = {"entry": kind, "dtype": "bf16", "T": 128, "K": rng.choice([5, 5, 5, 8]),
                "data": rng.choice(["lowrank", "gauss", "heavy"])}
        lo, hi, most = 64, 4096, 16
        if kind == "tiled":
            case["T"] = rng.choice([32, 64, 128, 128, 256])
        elif kind == "tiled32":
            case.update(entry="tiled", dtype="f32", T=rng.choice([32, 64, 128]))
        elif kind in ("gemm", "step_gemm"):
            case.update(entry="gemm" if kind == "gemm" else "step", T=rng.choice([512, 512, 0]))
            lo, most = 384, 8
        parts, left = [], _log_uniform(rng, 1, most)
        for i in range(min(left, rng.randint(1, 3))):
            h, w = (_log_uniform(rng, lo, hi) for _ in range(2))
            h, w = (max(64, 64 * round(d / 64)) if rng.random() < 0.5 else d for d in (h, w))
            n = left if i == 2 else rng.randint(1, left)
            left -= n
            parts.append(f"{n}*{h}x{w}")
            if left == 0:
                break
        case["shapes"] = ",".join(parts)
        if work(case)["flops"] <= (1.2e12 if case["dtype"] == "bf16" else 2.5e11):
            return case


def _matrix(shape, data, gen):
    H, W = shape
    if data == "lowrank":
        r = min(64, H, W)
        u = torch.randn(H, r, generator=gen, device="cuda") / math.sqrt(H)
        v = torch.randn(r, W, generator=gen, device="cuda") / math.sqrt(W)
        u /= torch.arange(1, r + 1, device="cuda", dtype=torch.float32)
        return torch.randn(H, W, generator=gen, device="cuda").mul_(0.01).addmm_(u, v)
    x = torch.randn(H, W, generator=gen, device="cuda")
    if data == "heavy":  # Student t with three degrees of freedom
        s = torch.zeros_like(x)
        for _ in range(3):
            s += torch.randn(H, W, generator=gen, device="cuda").square_()
        x.mul_(0.02).div_(s.div_(3.0).sqrt_())
    return x


_TYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _inputs(case, seed):
    """The gradients (or plain matrices); for a step also weights and momenta."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * seed + 17)
    dt = _TYPES[case["dtype"]]
    shapes = _shapes(case)
    g = [_matrix(s, case["data"], gen).to(dt) for s in shapes]
    if case["entry"] != "step":
        return g, None, None
    w = [(0.02 * torch.randn(*s, generator=gen, device="cuda")).to(dt) for s in shapes]
    m = [(3.0 * _matrix(s, case["data"], gen)).to(dt) for s in shapes]
    return g, w, m


def prepare(case, seed):
    g, w, m = _inputs(case, seed)
    state = {"case": case, "g": g}
    if case["entry"] == "step":
        opt = hm.HiMuon(w, T=case["T"], K=case["K"], coeffs=COEFFS, lr=LR, momentum=BETA, weight_decay=DECAY,
                        nesterov=True, scale_c=SCALE)
        for dst, src in zip(opt.moms, m):  # a run under way: the momenta are not zero
            dst.copy_(src)
        state["opt"] = opt
        return state
    state["out"] = [torch.empty_like(x) for x in g]
    if case["entry"] == "gemm":  # a program that runs one shape many times has its GEMMs tuned once
        hm.gemm_tune(_shapes(case), case["T"], hm.BF16, K=case["K"], coeffs=COEFFS)
    return state


def run(state):
    case = state["case"]
    if case["entry"] == "step":
        opt = state["opt"]
        return list(opt.step(state["g"])) + list(opt.moms)
    f = hm.ns_tiled if case["entry"] == "tiled" else hm.ns_gemm
    return f(state["g"], outputs=state["out"], T=case["T"], K=case["K"], coeffs=COEFFS)


def work(case):
    """Each matrix read and written once (a step: G, M, W read, M, W written).
    Per block of m x n (m <= n) and Newton-Schulz step: the symmetric A = X X^T
    and B = bA + cA^2 once per pair of entries, and B X in full."""
    size = 4 if case["dtype"] == "f32" else 2
    elems = flops = 0
    T = case["T"]
    for H, W in _shapes(case):
        elems += H * W
        th, tw = (H, W) if T == 0 or T >= max(H, W) else (T, T)
        for h, nh in ((th, H // th), (H % th, 1)):
            for w, nw in ((tw, W // tw), (W % tw, 1)):
                m, n = min(h, w), max(h, w)
                flops += nh * nw * (3 * m * m * n + m * m * m)
    return {"bytes": elems * size * (5 if case["entry"] == "step" else 2), "flops": flops * case["K"]}


def tolerance(case):
    """About four times the distance from fp64 that a pass shows: 0.6e-6 to
    1.3e-6 in fp32; 2.1e-3 to 3.2e-3 for a bf16 result from fp16 operands; 1.7e-3
    to 1.9e-3 for a step's weights and momenta, which bf16 rounding sets."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6}
    return {"rel": 8e-3 if case["entry"] == "step" else 1.2e-2}


def _phi(x, K):
    """Phi_K of a batch of blocks in fp64."""
    a, b, c = COEFFS
    tall = x.shape[1] > x.shape[2]
    if tall:
        x = x.transpose(1, 2).contiguous()
    n = x.flatten(1).norm(dim=1).clamp_min(1e-300)
    x = x / n[:, None, None]
    for _ in range(K):
        A = torch.bmm(x, x.transpose(1, 2))
        x = a * x + torch.bmm(b * A + c * torch.bmm(A, A), x)
    return x.transpose(1, 2) if tall else x


def _map(x, T, K):
    H, W = x.shape
    if T == 0 or T >= max(H, W):
        return _phi(x[None], K)[0]
    R, C = -(-H // T), -(-W // T)
    t = F.pad(x, (0, C * T - W, 0, R * T - H)).view(R, T, C, T).transpose(1, 2).reshape(R * C, T, T)
    y = torch.cat([_phi(p, K) for p in t.split(max(1, (1 << 26) // (T * T)))])
    return y.view(R, C, T, T).transpose(1, 2).reshape(R * T, C * T)[:H, :W]


def exact(case, seed):
    g, w, m = _inputs(case, seed)
    T, K = case["T"], case["K"]
    if case["entry"] != "step":
        return [_map(x.double(), T, K) for x in g]
    ws, ms = [], []
    for G, W, M in zip(g, w, m):
        G, W, M = G.double(), W.double(), M.double()
        M = BETA * M + G
        big = max(G.shape)
        tau = SCALE * math.sqrt(big if T == 0 or T >= big else T)
        ws.append((1.0 - LR * DECAY) * W - LR * tau * _map(G + BETA * M, T, K))
        ms.append(M)
    return ws + ms
