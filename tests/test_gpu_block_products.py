"""The block products of the large-tile path (ns_block_gemm.hip) against the
fp64 oracle, where they can go wrong: iterates that end inside a tile or a
64-column pad, each tile size that the launcher chooses by the number of
tiles, both operand types and both signs of c. Every tile size sums each
product in the same order, so a batch (large tiles) equals its matrices one by
one (small tiles) bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_27216_amd as hm
from parity import BF16_OPERAND_BAR, COEF32, to_f64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def rand(shape, seed):
    return torch.tensor(np.random.default_rng(seed).standard_normal(shape), dtype=torch.bfloat16).to(DEV)


def error(y, x, K, coeffs):
    r = oracle.phi_k(to_f64(x), K, *coeffs)
    return np.linalg.norm(to_f64(y) - r) / np.linalg.norm(r)


@pytest.mark.parametrize("shape,count", [
    ((256, 256), 1), ((257, 256), 1), ((256, 321), 1), ((300, 1000), 1), ((900, 449), 1),  # 64-tiles
    ((576, 640), 16), ((513, 700), 16),                                                     # 128-tiles
    ((1088, 1100), 8),                                                                      # 128 x 256 in B X
])
def test_whole_matrices(shape, count):
    print(f"[gpu-case] block products {count} x {shape}", flush=True)
    xs = [rand(shape, 10 * count + i) for i in range(count)]
    ys = hm.ns_gemm(xs, T=0, K=5, coeffs=COEF32)
    torch.cuda.synchronize()
    for i in {0, count - 1}:
        assert error(ys[i], xs[i], 5, COEF32) <= 1e-2  # fp16 operands, bf16 result: 2.1e-3 measured
        (alone,) = hm.ns_gemm([xs[i]], T=0, K=5, coeffs=COEF32)
        torch.cuda.synchronize()
        assert torch.equal(alone, ys[i])


@pytest.mark.parametrize("coeffs", [COEF32, (1.5, -0.5, -0.0625), (2.0, -1.5, 0.5)])
@pytest.mark.parametrize("compute", [hm.COMPUTE_DEFAULT, hm.COMPUTE_BF16])
def test_operands_and_signs(coeffs, compute):
    print(f"[gpu-case] block products coeffs={coeffs} compute={compute}", flush=True)
    coeffs = tuple(float(np.float32(v)) for v in coeffs)
    x = rand((330, 530), 5)
    (y,) = hm.ns_gemm([x], T=0, K=4, coeffs=coeffs, compute=compute)
    torch.cuda.synchronize()
    assert error(y, x, 4, coeffs) <= (BF16_OPERAND_BAR if compute == hm.COMPUTE_BF16 else 1e-2)


def test_budget_of_one_problem():
    """A chunk budget of exactly one unpadded problem is enough (its iterate is
    rounded up to 320 x 384), and chunking changes no bit."""
    print("[gpu-case] block products, chunk budget of one problem", flush=True)
    xs = [rand((257, 321), 40 + i) for i in range(3)]
    budget = (2 * 257 * 321 + 2 * 257 * 257) * 2
    one = hm.ns_gemm(xs, T=0, K=5, coeffs=COEF32, chunk_budget_bytes=budget)
    allin = hm.ns_gemm(xs, T=0, K=5, coeffs=COEF32)
    torch.cuda.synchronize()
    for a, b in zip(one, allin):
        assert torch.equal(a, b)
    with pytest.raises(hm.HimuonError):
        hm.ns_gemm(xs, T=0, K=5, coeffs=COEF32, chunk_budget_bytes=budget - 1)
