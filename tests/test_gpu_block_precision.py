"""How far the block products are from fp64, against an emulation that adds a X
in fp32 and rounds X, A and B once each to the operand type. A coefficient
rounded to 16 bits on the way (a I taken into the operand B) lies 8% (fp16
operands) to three times (bf16) above it. The distances are norms over 2e5
roundings and more, so two correct orders of summation agree to about 0.5%; the
bar is 3% above the emulation.
"""
import numpy as np
import pytest
import torch

import paper_2606_27216_amd as hm
from parity import COEF32

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def phi(x, K, coeffs):
    a, b, c = coeffs
    x = x.double() / x.double().norm()
    for _ in range(K):
        A = x @ x.T
        x = a * x + (b * A + c * (A @ A)) @ x
    return x


def emulated(x, K, coeffs, dtype):
    a, b, c = coeffs
    s2 = float(min(x.shape[0], 4096)) if dtype == torch.float16 else 1.0
    X = (x.double() * (s2**0.5 / x.double().norm())).float().to(dtype).float()
    for _ in range(K):
        A = (X @ X.T).to(dtype).float()
        B = ((c / s2**2) * (A @ A) + (b / s2) * A).to(dtype).float()
        X = (B @ X + a * X).to(dtype).float()
    return (X / s2**0.5).to(torch.bfloat16)


F16, BF16 = (hm.COMPUTE_DEFAULT, torch.float16), (hm.COMPUTE_BF16, torch.bfloat16)


@pytest.mark.parametrize("shape,coeffs,operand", [
    ((512, 512), COEF32, F16), ((300, 700), (1.875, -1.25, 0.375), F16), ((1024, 3000), (1.5, -0.5, -0.0625), F16),
    ((512, 512), COEF32, BF16), ((1024, 3000), (1.5, -0.5, -0.0625), BF16),
    ((512, 512), (3.3333, -0.01, 0.01), BF16),  # (its iterates leave fp16's range)
])
def test_distance_from_fp64(shape, coeffs, operand):
    compute, dtype = operand
    print(f"[gpu-case] block precision {shape} {coeffs} {dtype}", flush=True)
    coeffs = tuple(float(np.float32(v)) for v in coeffs)
    x = torch.tensor(np.random.default_rng(7).standard_normal(shape), dtype=torch.bfloat16).to(DEV)
    r = phi(x, 5, coeffs)
    (y,) = hm.ns_gemm([x], T=0, K=5, coeffs=coeffs, compute=compute)
    got = ((y.double() - r).norm() / r.norm()).item()
    bar = ((emulated(x, 5, coeffs, dtype).double() - r).norm() / r.norm()).item()
    print(f"error {got:.3e}, emulated {bar:.3e}", flush=True)
    assert got <= 1.03 * bar, (got, bar)


@pytest.mark.parametrize("shape", [(330, 530), (530, 330), (256, 256)])
def test_no_steps(shape):
    """K = 0: gather and scatter alone, through the panels: X / ||X||_F rounded to
    fp16 (11 bits) and bf16 (8 bits), at most 2^-11 and 2^-8 of the value (and, for
    fp16 subnormals, 2^-25 of the scaled iterate)."""
    print(f"[gpu-case] block products, no steps, {shape}", flush=True)
    x = torch.tensor(np.random.default_rng(8).standard_normal(shape), dtype=torch.bfloat16).to(DEV)
    (y,) = hm.ns_gemm([x], T=0, K=0, coeffs=COEF32)
    r = x.double() / x.double().norm()
    assert ((y.double() - r).abs() <= (2.0**-11 + 2.0**-8 + 2.0**-16) * r.abs() + 2.0**-25).all()
