"""fp32 32-tiles of small calls run on four waves per tile, those of large calls on
one: the results are the same bit for bit, across the line between them (512
tiles), for c != 0 and c = 0, ragged edges, K = 0 and in place."""
import pytest
import torch

import paper_2606_27216_amd as hm
from parity import COEF32

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("coeffs", [COEF32, (1.5, -0.5, 0.0), (2.0, -1.5, -0.5)])
@pytest.mark.parametrize("K", [0, 1, 5])
def test_split_equals_one_wave(coeffs, K):
    print(f"[gpu-case] split 32-tiles coeffs={coeffs} K={K}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(K)
    xs = [torch.randn(h, w, generator=g, device=DEV) for h, w in ((512, 512), (500, 511), (33, 1), (40, 70))]
    together = hm.ns_tiled(xs, T=32, K=K, coeffs=coeffs)  # 520 tiles
    alone = [hm.ns_tiled([x], T=32, K=K, coeffs=coeffs)[0] for x in xs]
    inplace = [x.clone() for x in xs]
    for x in inplace:
        hm.ns_tiled([x], [x], T=32, K=K, coeffs=coeffs)
    torch.cuda.synchronize()
    for a, b, c in zip(together, alone, inplace):
        assert torch.equal(a, b) and torch.equal(b, c)
