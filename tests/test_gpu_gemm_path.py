"""The library-GEMM path (himuon_ns_gemm) against the fp64 oracle.

T = 0 is Phi_K of the whole matrix (the full-matrix branch, Sec. 4.4.3):
checked against the oracle's phi_k, with the relative Frobenius error of the
whole matrix. T >= 1 is the tiled map with each tile a GEMM problem
(T = 512, the multi-kernel tile of Sec. 4.4.1): checked tile by tile against
the oracle's ns_tiled. Bars as for the fused kernels: 1e-5 (fp32 storage),
2e-2 (bf16 storage).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_27216_amd as hm
from parity import BF16_OPERAND_BAR, COEF32, TOL, tile_errors, to_f64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def announce(msg):
    print(f"[gpu-case] {msg}", flush=True)


def rand(shape, dtype, seed, scale=1.0):
    g = np.random.default_rng(seed)
    x = g.standard_normal(shape) * scale
    return torch.tensor(x, dtype=torch.float32).to(dtype).to(DEV)


def rel(y, r):
    nr = np.linalg.norm(r)
    return (0.0 if not np.any(y) else np.inf) if nr == 0 else np.linalg.norm(y - r) / nr


def gemm(mats, T, K=5, coeffs=COEF32, compute=hm.COMPUTE_DEFAULT, budget=0):
    out = hm.ns_gemm(mats, T=T, K=K, coeffs=coeffs, compute=compute, chunk_budget_bytes=budget)
    torch.cuda.synchronize()
    return out


SHAPES = [(384, 640), (640, 384), (512, 512), (1, 700), (333, 1), (257, 1000)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_full_matrix(dtype):
    announce(f"gemm T=0 dtype={dtype} shapes={SHAPES}")
    mats = [rand(s, dtype, 100 + i) for i, s in enumerate(SHAPES)]
    out = gemm(mats, T=0)
    for x, y in zip(mats, out):
        e = rel(to_f64(y), oracle.phi_k(to_f64(x), 5, *COEF32))
        assert e <= TOL[dtype], f"{tuple(x.shape)}: error {e:.3e}"


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_tiles_512(dtype):
    announce(f"gemm T=512 dtype={dtype} (ragged 2x2 tile grid)")
    x = rand((700, 900), dtype, 7)
    y = gemm([x], T=512)[0]
    R = oracle.ns_tiled(to_f64(x), 512, 5, *COEF32)
    e = tile_errors(to_f64(y), R, 512)
    assert e.max() <= TOL[dtype], f"max per-tile error {e.max():.3e}"


def test_tiles_128_agree_with_fused_kernel():
    announce("gemm T=128 vs oracle and vs the fused kernel, bf16")
    x = rand((384, 520), torch.bfloat16, 11)
    y = gemm([x], T=128)[0]
    z = hm.ns_tiled([x], T=128, K=5, coeffs=COEF32)[0]
    torch.cuda.synchronize()
    R = oracle.ns_tiled(to_f64(x), 128, 5, *COEF32)
    assert tile_errors(to_f64(y), R, 128).max() <= 2e-2
    assert tile_errors(to_f64(y), to_f64(z), 128).max() <= 2e-2


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_zero_and_k0(dtype):
    announce(f"gemm zero matrix and K=0, dtype={dtype}")
    z = torch.zeros((200, 300), dtype=dtype, device=DEV)
    assert not torch.any(gemm([z], T=0)[0])
    x = rand((200, 300), dtype, 3, scale=1e3)
    y0 = gemm([x], T=0, K=0)[0]
    S = to_f64(x)
    assert rel(to_f64(y0), S / np.linalg.norm(S)) <= TOL[dtype]


def test_chunked_matches_one_chunk():
    announce("gemm T=512 with several chunks vs one chunk, bf16")
    mats = [rand((1024, 1024), torch.bfloat16, 40 + i) for i in range(2)]
    one = gemm(mats, T=512)
    ws1 = hm.himuon_ns_gemm_workspace_size([1024, 1024], [1024, 1024], 512, hm.BF16, 0, 5, *COEF32)
    per = 2 * (2 * 512 * 512 + 2 * 512 * 512)  # fp16 iterate buffers of one problem
    many = gemm(mats, T=512, budget=3 * per)
    ws3 = hm.himuon_ns_gemm_workspace_size([1024, 1024], [1024, 1024], 512, hm.BF16, 0, 5, *COEF32, 3 * per)
    assert ws3 < ws1
    for a, b, x in zip(one, many, mats):
        R = oracle.ns_tiled(to_f64(x), 512, 5, *COEF32)
        assert tile_errors(to_f64(a), R, 512).max() <= 2e-2
        assert tile_errors(to_f64(b), R, 512).max() <= 2e-2
        assert tile_errors(to_f64(a), to_f64(b), 512).max() <= 1e-3


def test_transpose_equivariance():
    announce("gemm T=0: Phi(S^T) = Phi(S)^T, fp32")
    x = rand((300, 500), torch.float32, 5)
    y = gemm([x], T=0)[0]
    yt = gemm([x.t().contiguous()], T=0)[0]
    assert rel(to_f64(yt).T, to_f64(y)) <= 2e-6


def test_tuned_kernels_match_oracle():
    """gemm_tune on calls that the block products serve (nothing to pick: it
    returns) and their results (T = 512 tiles and whole matrices). Calls whose
    candidates are timed are in test_gpu_library_products.py."""
    announce("gemm tune, then T=512 and T=0 vs oracle, bf16")
    x = rand((700, 900), torch.bfloat16, 17)
    hm.gemm_tune([(700, 900)], 512, hm.BF16, K=5, coeffs=COEF32)
    hm.gemm_tune([(700, 900)], 0, hm.BF16, K=5, coeffs=COEF32)
    torch.cuda.synchronize()
    y = gemm([x], T=512)[0]
    e = tile_errors(to_f64(y), oracle.ns_tiled(to_f64(x), 512, 5, *COEF32), 512)
    assert e.max() <= 2e-2, f"T=512: {e.max():.3e}"
    y0 = gemm([x], T=0)[0]
    e0 = rel(to_f64(y0), oracle.phi_k(to_f64(x), 5, *COEF32))
    assert e0 <= 2e-2, f"T=0: {e0:.3e}"


RECT = [(256, 128), (128, 512), (64, 1024), (512, 96)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_rectangular_tiles(dtype):
    """T_h x T_w tiles (the tile-shape study) against the oracle's rectangular
    tiling, tile by tile; tall tiles go through the orientation rule."""
    x = rand((700, 900), dtype, 23)
    for Th, Tw in RECT:
        announce(f"gemm rectangular tiles {Th}x{Tw} dtype={dtype} on 700x900")
        y = hm.ns_gemm([x], T=Th, Tw=Tw, K=5, coeffs=COEF32)[0]
        torch.cuda.synchronize()
        R = oracle.ns_tiled_hw(to_f64(x), Th, Tw, 5, *COEF32)
        Y = to_f64(y)
        worst = 0.0
        for r0 in range(0, 700, Th):
            for c0 in range(0, 900, Tw):
                sl = np.s_[r0:r0 + Th, c0:c0 + Tw]
                worst = max(worst, rel(Y[sl], R[sl]))
        assert worst <= TOL[dtype], f"{Th}x{Tw}: max per-tile error {worst:.3e}"


def test_rectangular_square_and_covering_tiles():
    """Th = Tw reproduces the square call bit for bit; one tile covering the
    matrix is the full map."""
    announce("gemm rectangular: square case and a covering tile, bf16")
    x = rand((300, 500), torch.bfloat16, 29)
    a = hm.ns_gemm([x], T=128, K=5, coeffs=COEF32)[0]
    b = hm.ns_gemm([x], T=128, Tw=128, K=5, coeffs=COEF32)[0]
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    y = hm.ns_gemm([x], T=512, Tw=600, K=5, coeffs=COEF32)[0]
    torch.cuda.synchronize()
    assert rel(to_f64(y), oracle.phi_k(to_f64(x), 5, *COEF32)) <= 2e-2


@pytest.mark.parametrize("dtype,compute", [(torch.float32, hm.COMPUTE_DEFAULT), (torch.bfloat16, hm.COMPUTE_BF16)])
def test_tiles_256_where_no_fused_kernel_exists(dtype, compute):
    """T = 256 with fp32 storage, or with bf16 operands, has no fused kernel
    (the tile does not fit one CU's LDS in those forms): himuon_ns_tiled runs
    such a call on the GEMM path, so it equals himuon_ns_gemm at T = 256 bit
    for bit, and both meet the oracle's bar."""
    announce(f"gemm T=256 dtype={dtype} compute={compute}")
    x = rand((600, 700), dtype, 31)
    y = gemm([x], T=256, compute=compute)[0]
    z = hm.ns_tiled([x], T=256, K=5, coeffs=COEF32, compute=compute)[0]
    torch.cuda.synchronize()
    assert torch.equal(y, z)
    e = tile_errors(to_f64(y), oracle.ns_tiled(to_f64(x), 256, 5, *COEF32), 256)
    print(f"[gpu-err] 600x700 T=256 {dtype}: max {e.max():.3e}", flush=True)
    assert e.max() <= (TOL[dtype] if compute != hm.COMPUTE_BF16 else BF16_OPERAND_BAR), \
        f"max per-tile error {e.max():.3e}"


@pytest.mark.parametrize("shape", [(6144, 8192), (8192, 6144)])
def test_full_matrix_large_gram_closed_form(shape):
    """Whole matrices with a Gram size above 4096, where the fp16 iterate
    scale is capped (s^2 = 4096 instead of m), checked against the SVD
    closed form: S = P D Q with P, Q permutations and D diagonal has singular
    values d, so Phi_K(S) = P p^K(D / ||D||_F) Q, with p the scalar map
    s -> a s + b s^3 + c s^5 (too large for the fp64 oracle in test time)."""
    H, W = shape
    announce(f"gemm T=0 bf16 {H}x{W} permuted diagonal, closed form")
    m = min(H, W)
    g = np.random.default_rng(H + W)
    d = np.exp(g.uniform(np.log(1e-3), 0.0, m))
    rows = g.permutation(H)[:m]
    cols = g.permutation(W)[:m]
    S = torch.zeros((H, W), dtype=torch.float32)
    S[torch.as_tensor(rows), torch.as_tensor(cols)] = torch.as_tensor(d, dtype=torch.float32)
    x = S.to(torch.bfloat16).to(DEV)
    y = gemm([x], T=0)[0]
    dv = to_f64(x)[rows, cols]  # the stored (bf16) values
    s = dv / np.linalg.norm(dv)
    a, b, c = COEF32
    for _ in range(5):
        s = a * s + b * s ** 3 + c * s ** 5
    Y = to_f64(y)
    got = Y[rows, cols]
    off = Y.copy()
    off[rows, cols] = 0.0
    err = np.sqrt(np.sum((got - s) ** 2) + np.sum(off ** 2)) / np.linalg.norm(s)
    print(f"[gpu-err] {H}x{W} closed form: {err:.3e}", flush=True)
    assert err <= TOL[torch.bfloat16], err


@pytest.mark.parametrize("T", [512, 0])
def test_in_place_equals_out_of_place(T):
    """out == in (allowed, as for himuon_ns_tiled): each chunk gathers all of
    its blocks before it scatters any, and blocks of different problems do
    not overlap, so the result is the out-of-place one, bit for bit."""
    announce(f"gemm in place, T={T}, bf16, several chunks")
    mats = [rand((700, 900), torch.bfloat16, 61), rand((1024, 512), torch.bfloat16, 62)]
    budget = 2 * (2 * 512 * 512 + 2 * 512 * 512) * 2 if T else 0  # two 512-tiles per chunk
    ref = hm.ns_gemm(mats, T=T, K=5, coeffs=COEF32, chunk_budget_bytes=budget)
    inplace = [m.clone() for m in mats]
    hm.ns_gemm(inplace, outputs=inplace, T=T, K=5, coeffs=COEF32, chunk_budget_bytes=budget)
    torch.cuda.synchronize()
    for a, b in zip(ref, inplace):
        assert torch.equal(a, b)
