"""The last block product of an optimizer step writes the weights itself: every
tile size that the launcher chooses, wide matrices and transposed ones, against
fp64 on the device. With W = 0 and no decay the step leaves -lr tau U, so U itself
is compared; the same step with weights and decay, up to one bf16 rounding of W.
"""
import pytest
import torch

import paper_2606_27216_amd as hm
from parity import COEF32
from test_gpu_library_products import phi, rand

pytestmark = pytest.mark.gpu

LR, SC, WD = 0.1, 0.2, 0.5


@pytest.mark.parametrize("shape,count", [((300, 500), 1), ((500, 300), 1),        # 64-tiles
                                         ((600, 1000), 8), ((1000, 600), 8),      # 128-tiles
                                         ((1088, 2100), 8), ((2100, 1088), 8)])   # 128 x 256
@pytest.mark.parametrize("nesterov", [True, False])
def test_step_whole(shape, count, nesterov):
    print(f"[gpu-case] block products into weights {count} x {shape} nesterov={nesterov}", flush=True)
    bf = torch.bfloat16
    gs = [rand(shape, bf, 10 + i) for i in range(count)]
    ms = [rand(shape, bf, 30 + i) for i in range(count)]
    ws = [0.05 * rand(shape, bf, 50 + i) for i in range(count)]
    tau = SC * max(shape) ** 0.5
    opts = dict(T=0, K=5, coeffs=COEF32, lr=LR, momentum=0.5, nesterov=nesterov, scale_c=SC)
    zero = [torch.zeros_like(w) for w in ws]
    m0 = [m.clone() for m in ms]
    hm.step(zero, gs, m0, weight_decay=0.0, **opts)
    w1, m1 = [w.clone() for w in ws], [m.clone() for m in ms]
    hm.step(w1, gs, m1, weight_decay=WD, **opts)
    for i in {0, count - 1}:
        m = 0.5 * ms[i].double() + gs[i].double()
        assert ((m0[i].double() - m).abs() <= 2.0**-8 * m.abs() + 1e-6).all() and torch.equal(m0[i], m1[i])
        m = m0[i].double()
        u = LR * tau * phi(gs[i].double() + 0.5 * m if nesterov else m, 5, COEF32)
        # fp16 operands and the bf16 store: 2.2e-3 measured on the map
        assert ((zero[i].double() + u).norm() / u.norm()).item() <= 1e-2
        r = (1.0 - LR * WD) * ws[i].double() - u
        err = (w1[i].double() - r).abs()
        assert err.norm() <= 1e-2 * u.norm() + 2.0**-8 * r.norm()
        # nothing is missing or out of place: no entry is off by the size of an update
        assert err.max() <= 0.2 * u.abs().max() + 2.0**-8 * r.abs().max()
