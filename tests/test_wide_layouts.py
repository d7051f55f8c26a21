"""The wide tiles of the layouts B stored N x K and A stored K x M: exact on small integers at their
edges, in the CPU model of the hardware and on the GPU."""
import numpy as np
import pytest
import torch

import emu_util as emu
import oracle
import paper_2210_16691_amd as al
import workloads as wl

CODE = {"f16": al.F16, "bf16": al.BF16}
ODT = {"f16": oracle.F16, "bf16": oracle.BF16}
WIDE = [((256, 256, 32, 128, 64), 0, 1), ((256, 128, 64, 128, 64), 0, 1), ((256, 192, 32, 128, 96), 1, 0),
        ((256, 128, 64, 128, 64), 1, 0)]


def _operands(M, N, K, dt, tA, tB):
    A = wl.small_ints((K, M) if tA else (M, K), dt, 9900 + M)
    B = wl.small_ints((N, K) if tB else (K, N), dt, 9901 + N)
    return A, B, oracle.gemm(wl.bits(A), wl.bits(B), ODT[dt], bool(tA), bool(tB))


@pytest.mark.parametrize("tile,tA,tB", [WIDE[0], WIDE[2]])
def test_on_the_cpu_model(tile, tA, tB):
    for n, (M, N, K) in enumerate([(264, 200, 136), (8, 8, 32)]):
        A, B, ref = _operands(M, N, K, "bf16", tA, tB)
        C = torch.full((M, N), float("nan"))
        errs = emu.call(al.alcop_gemm, A, B, C, al.sched(*tile, 3, 2, 1), bool(tB), transA=bool(tA), reads=[A, B],
                        writes=[C], policy=emu.POLICIES[n])
        assert not errs, (M, N, K, errs[:4])
        assert np.array_equal(C.double().numpy(), ref), (M, N, K)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("tile,tA,tB", WIDE)
def test_on_the_gpu(tile, tA, tB, dt):
    for M, N, K in [(264, 200, 136), (8, 8, 32), (1040, 776, 520)]:
        A, B, ref = _operands(M, N, K, dt, tA, tB)
        ran = 0
        for stages in (3, 4):
            s = al.sched(*tile, stages, 2, 1)
            prob = al.problem(al.OP_GEMM, M, N, K, CODE[dt], al.F32, transA=tA, transB=tB)
            if al.alcop_sched_supported(prob, s) != al.OK:       # four stages of the larger tiles do not fit
                continue
            C = torch.full((M, N), float("nan"), device="cuda")
            al.alcop_gemm(A.cuda(), B.cuda(), C, s, bool(tB), transA=bool(tA))
            torch.cuda.synchronize()
            assert np.array_equal(C.cpu().double().numpy(), ref), (M, N, K, stages)
            ran += 1
        assert ran


@pytest.mark.gpu
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dt", ["f16", "bf16"])
def test_default_pick_on_the_gpu(dt, tA, tB):
    # few tiles, one turn of the machine, several: every kind of kernel the pick knows
    for M, N, K in [(16, 64, 1032), (264, 520, 4104), (1032, 2008, 136), (2056, 3080, 264), (5000, 776, 72)]:
        A, B, ref = _operands(M, N, K, dt, tA, tB)
        C = torch.full((M, N), float("nan"), device="cuda")
        al.alcop_gemm(A.cuda(), B.cuda(), C, None, bool(tB), transA=bool(tA))
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().double().numpy(), ref), (M, N, K)
