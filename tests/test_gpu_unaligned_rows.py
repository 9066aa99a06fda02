"""Rows that are not 16-byte aligned and chunks that the last column cuts
(every remainder of eight columns), at each tile size and storage type: the
result equals, bit for bit, that of the same values in an aligned, padded
buffer, in place and out of place, and nothing outside the matrix is written.
"""
import pytest
import torch

import paper_2606_27216_amd as hm
from parity import COEF32

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T", [32, 64, 128, 256, 512])
def test_odd_rows_equal_aligned_rows(T, dtype):
    print(f"[gpu-case] unaligned rows T={T} {dtype}", flush=True)
    f = hm.ns_gemm if T == 512 else hm.ns_tiled
    for i, (h, w) in enumerate([(33, 129 + r) for r in range(8)] + [(40, 5), (3, 7), (130, 261)]):
        g = torch.Generator(device=DEV)
        g.manual_seed(100 * T + i)
        x = torch.randn(h, w, generator=g, device=DEV).to(dtype)
        pitch = (w + 15) // 8 * 8
        aligned = torch.zeros(h, pitch, dtype=dtype, device=DEV)[:, :w].copy_(x)
        (ref,) = f([aligned], [torch.zeros(h, pitch, dtype=dtype, device=DEV)[:, :w]], T=T, K=3, coeffs=COEF32)
        for ld, shift in ((w, 0), (w + 3, 1), (w + 2, 5)):  # odd pitch, odd base
            buf = torch.full((shift + h * ld + 8,), 7.0, dtype=dtype, device=DEV)
            view = buf[shift:shift + h * ld].view(h, ld)[:, :w]
            view.copy_(x)
            out = torch.full_like(buf, 7.0)
            oview = out[shift:shift + h * ld].view(h, ld)[:, :w]
            f([view], [oview], T=T, K=3, coeffs=COEF32)
            torch.cuda.synchronize()
            assert torch.equal(oview, ref), (h, w, ld)
            oview.fill_(7.0)
            assert bool((out == 7.0).all()), (h, w, ld)
            f([view], [view], T=T, K=3, coeffs=COEF32)
            torch.cuda.synchronize()
            assert torch.equal(view, ref), (h, w, ld)
