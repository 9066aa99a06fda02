"""fp16-operand tiles of 128 and 256 run on kernels with and without code for cut
or unaligned tiles, and in calls that hold both kinds on one kernel with both tile
loops (step; map from 8192 whole tiles on), whole matrices first: a matrix has
the same bits alone and beside others, whatever the kernel, the order and the
chunks; the step on whole matrices agrees with the oracle.
"""
import pytest
import torch

import paper_2606_27216_amd as hm
from parity import COEF32
from test_gpu_step import BETA, LR, SC, WD, W_SCALE, check_step, rand

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
COEFFS = [COEF32, (1.5, -0.5, -0.0625), (1.5, -0.5, 0.0)]  # c > 0, c < 0, c = 0


@pytest.mark.parametrize("coeffs", COEFFS)
@pytest.mark.parametrize("T", [128, 256])
def test_map_beside_cut_matrices(T, coeffs):
    print(f"[gpu-case] whole beside cut T={T} coeffs={coeffs}", flush=True)
    shapes = [(300, 421), (2 * T, 3 * T), (T, T), (33, 1001), (4 * T, T), (T, 5 * T + 8)]
    xs = [rand(s, torch.bfloat16, 10 + i, 1.0) for i, s in enumerate(shapes)]
    alone = [hm.ns_tiled([x], T=T, K=5, coeffs=coeffs)[0] for x in xs]
    for budget in (0, 5 * 2 * T * T * 2):
        for a, b in zip(alone, hm.ns_tiled(xs, T=T, K=5, coeffs=coeffs, chunk_budget_bytes=budget)):
            assert torch.equal(a, b)
    # a whole matrix whose rows are unaligned in memory is none
    buf = torch.zeros(2 * T, 3 * T + 1, dtype=torch.bfloat16, device=DEV)
    view = buf[:, :3 * T].copy_(xs[1])
    y, _ = hm.ns_tiled([view, xs[1]], T=T, K=5, coeffs=coeffs)
    assert torch.equal(y, alone[1])


@pytest.mark.parametrize("coeffs", COEFFS)
def test_map_of_both_loops(coeffs):
    print(f"[gpu-case] map of 8193 whole tiles beside cut ones, coeffs={coeffs}", flush=True)
    big = rand((4096, 4096), torch.bfloat16, 20, 1.0)
    odd = [rand(s, torch.bfloat16, 21 + i, 1.0) for i, s in enumerate([(333, 1001), (5, 9)])]
    small = rand((128, 128), torch.bfloat16, 23, 1.0)
    xs = odd + [big] * 4 + [small] + [big] * 4
    ys = hm.ns_tiled(xs, T=128, K=5, coeffs=coeffs)
    for x in (odd[0], odd[1], big, small):
        (alone,) = hm.ns_tiled([x], T=128, K=5, coeffs=coeffs)
        for i, z in enumerate(xs):
            if z is x:
                assert torch.equal(ys[i], alone), i


def test_tables_of_many_matrices():
    """More matrices than ride in the arguments: the table in a workspace and the
    one that upload kernels write both follow the order of the tiles."""
    print("[gpu-case] 100 matrices, whole and cut in turn", flush=True)
    xs = [rand((256, 128) if i % 3 else (100, 131), torch.bfloat16, 30 + i, 1.0) for i in range(100)]
    ys = hm.ns_tiled(xs, T=128, K=3, coeffs=COEF32)
    zs = [torch.empty_like(x) for x in xs]
    st = hm.himuon_ns_tiled_noalloc(
        len(xs), [x.data_ptr() for x in xs], [z.data_ptr() for z in zs], [x.shape[0] for x in xs],
        [x.shape[1] for x in xs], [x.stride(0) for x in xs], [z.stride(0) for z in zs], T=128, K=3, a=COEF32[0],
        b=COEF32[1], c=COEF32[2], dtype=hm.BF16, compute=hm.COMPUTE_DEFAULT, chunk_budget_bytes=0,
        stream=torch.cuda.current_stream().cuda_stream)
    assert st == hm.OK
    torch.cuda.synchronize()
    for i, x in enumerate(xs):
        (alone,) = hm.ns_tiled([x], T=128, K=3, coeffs=COEF32)
        assert torch.equal(ys[i], alone) and torch.equal(zs[i], alone), i


@pytest.mark.parametrize("count", [1, 9])
@pytest.mark.parametrize("nesterov", [True, False])
def test_step_whole_alone_and_beside_cut(nesterov, count):
    """(256, 384) and (1024, 512) alone: the kernel without edge code, against the
    oracle; beside cut matrices (27 and more tables: not in the arguments): the
    same bits, and the cut ones as in a call of their own."""
    print(f"[gpu-case] step whole tiles nesterov={nesterov} count={count}", flush=True)
    whole, cut = [(256, 384), (1024, 512)], [(333, 1001), (130, 128)]

    def step(shapes):
        ws = [rand(s, torch.bfloat16, 40 + s[0], W_SCALE) for s in shapes]
        gs = [rand(s, torch.bfloat16, 50 + s[0], 1e-2) for s in shapes]
        ms = [rand(s, torch.bfloat16, 60 + s[0], 1e-2) for s in shapes]
        w1, m1 = [w.clone() for w in ws], [m.clone() for m in ms]
        hm.step(w1, gs, m1, T=128, K=5, coeffs=COEF32, lr=LR, momentum=BETA, weight_decay=WD, nesterov=nesterov,
                scale_c=SC)
        torch.cuda.synchronize()
        return ws, gs, ms, w1, m1

    alone = step(whole)
    for w0, g, m0, w1, m1 in zip(*alone):
        check_step(w0, g, m0, w1, m1, 128, torch.bfloat16, LR, BETA, WD, nesterov, SC)
    ragged = step(cut)
    both = step((cut[:1] + whole + cut[1:]) * count)
    for i in range(count):
        for k in (3, 4):
            c0, a0, a1, c1 = both[k][4 * i:4 * i + 4]
            assert torch.equal(a0, alone[k][0]) and torch.equal(a1, alone[k][1])
            assert torch.equal(c0, ragged[k][0]) and torch.equal(c1, ragged[k][1])
