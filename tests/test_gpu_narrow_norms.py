"""Whole matrices that are narrow in one direction: norm passes whose parts begin
and end inside a row, and iterates on both sides of the line up to which the
block products serve a problem; coefficients whose c is too small to divide by.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_27216_amd as hm
from parity import COEF32, to_f64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("shape", [(1, 20001), (20001, 1), (7, 30011), (30011, 7), (64, 20000), (20000, 64), (9, 17)])
def test_normalised_block(shape, dtype):
    """K = 0 returns X / ||X||_F. fp32: half an ulp each of the factor and the
    product, tolerance 4 ulp. bf16: roundings to fp16 (11 bits) and to bf16 (8 bits),
    at most 2^-11 and 2^-8 of the value."""
    print(f"[gpu-case] norm of {shape} {dtype}", flush=True)
    x = torch.tensor(np.random.default_rng(3).uniform(0.5, 1.0, shape), dtype=dtype).to(DEV)
    (y,) = hm.ns_gemm([x], T=0, K=0)
    r = x.double() / x.double().norm()
    tol = 2.0**-21 if dtype == torch.float32 else 2.0**-11 + 2.0**-8 + 2.0**-16
    assert ((y.double() - r).abs() <= tol * r).all()
    # nothing of the sum is missing: roundings average out over the block
    if x.numel() > 1000:
        assert abs((y.double() * r).sum().item() - 1.0) <= (1e-6 if dtype == torch.float32 else 2e-3)


@pytest.mark.parametrize("shape", [(30011, 7), (7, 30011)])
def test_momentum_updated_once(shape):
    print(f"[gpu-case] momentum of {shape}", flush=True)
    rng = np.random.default_rng(4)
    w, g, m = (torch.tensor(rng.standard_normal(shape), dtype=torch.float32).to(DEV) for _ in range(3))
    r = 0.5 * m.double() + g.double()
    hm.step([w], [g], [m], T=0, K=1, lr=0.1, momentum=0.5, weight_decay=0.0, nesterov=False, scale_c=0.2)
    assert torch.allclose(m.double(), r, rtol=0, atol=1e-6)


def test_smallest_c():
    """b and c that vanish beside a: Phi_K is a^K X / ||X||_F."""
    print("[gpu-case] coefficients (1.5, -1e-30, 1e-42)", flush=True)
    x = torch.tensor(np.random.default_rng(5).standard_normal((330, 530)), dtype=torch.bfloat16).to(DEV)
    (y,) = hm.ns_gemm([x], T=0, K=2, coeffs=(1.5, -1e-30, 1e-42))
    r = 2.25 * x.double() / x.double().norm()
    assert ((y.double() - r).norm() / r.norm()).item() <= 1e-2


@pytest.mark.parametrize("shape", [(64, 4096), (64, 4097), (4097, 100), (1023, 4160)])
def test_long_iterates(shape):
    print(f"[gpu-case] long iterate {shape}", flush=True)
    x = torch.tensor(np.random.default_rng(6).standard_normal(shape), dtype=torch.bfloat16).to(DEV)
    (y,) = hm.ns_gemm([x], T=0, K=5, coeffs=COEF32)
    r = oracle.phi_k(to_f64(x), 5, *COEF32)
    assert np.linalg.norm(to_f64(y) - r) <= 1e-2 * np.linalg.norm(r)  # fp16 operands, bf16 result: 2.1e-3 measured
