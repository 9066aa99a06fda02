"""The calls whose products stay with the GEMM library: fp32 storage, c = 0,
iterates of few rows and long ones. Tuned; in one call with a group of the block
products (plan creation, the shared workspace, the tuner passing the other group
by); and from several host threads, which share the library's per-device handle
and plans. References in fp64 on the device.
"""
import threading

import pytest
import torch

import paper_2606_27216_amd as hm
from parity import COEF32

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
LINEAR = (1.5, -0.5, 0.0)
BAR = {torch.float32: 1e-5, torch.bfloat16: 1e-2}  # whole-matrix bars of the library path: 2.3e-6 and 2.2e-3 measured


def rand(shape, dtype, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn(*shape, generator=g, device=DEV).to(dtype)


def phi(x, K, coeffs):
    a, b, c = coeffs
    x = x.double() / x.double().norm()
    if x.shape[0] > x.shape[1]:
        return phi(x.t(), K, coeffs).t()
    for _ in range(K):
        A = x @ x.t()
        x = a * x + (b * A + c * (A @ A)) @ x
    return x


def check(ys, xs, coeffs):
    for y, x in zip(ys, xs):
        r = phi(x, 5, coeffs)
        assert ((y.double() - r).norm() / r.norm()).item() <= BAR[x.dtype], (tuple(x.shape), x.dtype)


CALLS = [  # (shapes, dtype, coefficients)
    ([(700, 900), (900, 700)], torch.float32, COEF32),
    ([(700, 900)], torch.bfloat16, LINEAR),
    ([(64, 8192), (20, 700)], torch.bfloat16, COEF32),
    ([(64, 8192), (700, 900), (300, 300), (20, 700)], torch.bfloat16, COEF32),  # library, block products, both again
]


@pytest.mark.parametrize("shapes,dtype,coeffs", CALLS)
def test_tuned_calls(shapes, dtype, coeffs):
    print(f"[gpu-case] library products, tuned: {shapes} {dtype} {coeffs}", flush=True)
    xs = [rand(s, dtype, 10 + i) for i, s in enumerate(shapes)]
    check(hm.ns_gemm(xs, T=0, K=5, coeffs=coeffs), xs, coeffs)
    hm.gemm_tune(shapes, 0, hm.F32 if dtype == torch.float32 else hm.BF16, K=5, coeffs=coeffs)
    check(hm.ns_gemm(xs, T=0, K=5, coeffs=coeffs), xs, coeffs)


def test_threads():
    """Four threads on their own streams, each with calls of its own shapes: the bits
    of the same calls made alone."""
    print("[gpu-case] library products from four threads", flush=True)
    calls = [([rand(s, dtype, 40 + 10 * n + i) for i, s in enumerate(shapes)], coeffs)
             for n, (shapes, dtype, coeffs) in enumerate(CALLS)]
    alone = [hm.ns_gemm(xs, T=0, K=5, coeffs=c) for xs, c in calls]
    torch.cuda.synchronize()
    results, errors = [None] * len(calls), []

    def worker(t):
        try:
            s = torch.cuda.Stream(device=DEV)
            xs, c = calls[t]
            for _ in range(6):
                out = hm.ns_gemm(xs, T=0, K=5, coeffs=c, stream=s)
            s.synchronize()
            results[t] = out
        except Exception as e:  # reported below, on the test's thread
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(t,)) for t in range(len(calls))]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not errors, errors
    for got, ref in zip(results, alone):
        for y, r in zip(got, ref):
            assert torch.equal(y, r)
