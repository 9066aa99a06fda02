"""The optimizer step on weights, gradients and momenta whose rows are not 16-byte
aligned and whose last chunks are cut (every remainder of eight columns): the bits
of the same step on aligned, padded buffers, and nothing outside the matrices is
written.
"""
import pytest
import torch

import paper_2606_27216_amd as hm
from parity import COEF32

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def padded(x, ld, shift):
    """x in a buffer of sevens with rows of `ld` elements from element `shift` on."""
    h, w = x.shape
    buf = torch.full((shift + h * ld + 8,), 7.0, dtype=x.dtype, device=DEV)
    view = buf[shift:shift + h * ld].view(h, ld)[:, :w]
    view.copy_(x)
    return buf, view


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T", [32, 64, 128, 256, 512])
def test_odd_rows_equal_aligned_rows(T, dtype):
    print(f"[gpu-case] unaligned step T={T} {dtype}", flush=True)
    opts = dict(T=T, K=3, coeffs=COEF32, lr=0.1, momentum=0.9, weight_decay=0.1, nesterov=True, scale_c=0.2)
    for i, (h, w) in enumerate([(33, 129 + r) for r in range(8)] + [(40, 5), (130, 261)]):
        g = torch.Generator(device=DEV)
        g.manual_seed(100 * T + i)
        src = [torch.randn(h, w, generator=g, device=DEV).to(dtype) for _ in range(3)]
        pitch = (w + 15) // 8 * 8
        ref = [padded(x, pitch, 0)[1] for x in src]
        hm.step([ref[0]], [ref[1]], [ref[2]], **opts)
        for ld, shift in ((w, 0), (w + 3, 1), (w + 2, 5)):  # odd pitch, odd base
            got = [padded(x, ld, shift) for x in src]
            hm.step([got[0][1]], [got[1][1]], [got[2][1]], **opts)
            torch.cuda.synchronize()
            for (buf, view), r in zip(got, ref):
                assert torch.equal(view, r), (h, w, ld)
                view.fill_(7.0)
                assert bool((buf == 7.0).all()), (h, w, ld)
