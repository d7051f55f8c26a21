"""Kernels whose waves split the reduction axis (schedule variant 3): exact on small integers at the
edges of tiles, k-tiles and wave slices, in the CPU model of the hardware and on the GPU."""
import numpy as np
import pytest
import torch

import emu_util as emu
import oracle
import paper_2210_16691_amd as al
import workloads as wl

TDT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
ADT = {"f16": al.F16, "bf16": al.BF16, "f32": al.F32}
ODT = {"f16": oracle.F16, "bf16": oracle.BF16}


def _sched(t):
    return al.sched(t[0], t[1], 64, t[0], t[1], t[2], 1, 0, 1, 0, 3)


# (tile, dt, transA, transB): what the CPU model holds of the kernels
EMU = [((16, 16, 2), "f16", 0, 0), ((16, 16, 2), "f16", 0, 1), ((16, 32, 2), "f16", 0, 0), ((16, 32, 2), "bf16", 0, 1),
       ((32, 32, 2), "f16", 0, 0), ((32, 32, 2), "f16", 1, 1), ((16, 16, 2), "bf16", 1, 0), ((32, 64, 2), "f16", 0, 0),
       ((32, 64, 2), "bf16", 1, 1)]
# one k-tile for eight waves, one each, a partial last k-tile, slices of unequal length; M and N
# below, at and just past a tile
SHAPES = [(1, 8, 8), (16, 16, 64), (17, 40, 520), (40, 24, 1096), (65, 72, 200)]


def _problem(M, N, K, dt, tA, tB, b=1):
    if tA:
        M = (M + 7) // 8 * 8
    sh = (lambda r, c: (b, r, c)) if b > 1 else (lambda r, c: (r, c))
    A = wl.small_ints(sh(K, M) if tA else sh(M, K), dt, 9300 + M)
    B = wl.small_ints(sh(N, K) if tB else sh(K, N), dt, 9400 + N)
    ref = (oracle.bmm if b > 1 else oracle.gemm)(wl.bits(A), wl.bits(B), ODT[dt], bool(tA), bool(tB))
    return M, A, B, ref


@pytest.mark.parametrize("tile,dt,tA,tB", EMU)
def test_matrix_kernels_on_the_cpu_model(tile, dt, tA, tB):
    for n, (M, N, K) in enumerate(SHAPES):
        M, A, B, ref = _problem(M, N, K, dt, tA, tB)
        C = torch.full((M, N), float("nan"))
        errs = emu.call(al.alcop_gemm, A, B, C, _sched(tile), bool(tB), transA=bool(tA), reads=[A, B], writes=[C],
                        policy=emu.POLICIES[n % 4])
        assert not errs, (M, N, K, errs[:4])
        assert np.array_equal(C.double().numpy(), ref), (M, N, K)


@pytest.mark.parametrize("mutation", [1, 3, 4])
def test_planted_synchronisation_mistakes_are_noticed(mutation):
    M, A, B, ref = _problem(40, 24, 1096, "f16", 0, 0)
    C = torch.full((M, 24), float("nan"))
    errs = emu.call(al.alcop_gemm, A, B, C, _sched((16, 16, 2) if mutation != 4 else (32, 32, 2)), reads=[A, B],
                    writes=[C], policy=(1, 0), mutation=mutation)
    assert errs or not np.array_equal(C.double().numpy(), ref)


CONVS = [((16, 16, 2), "f16", 0, (1, 5, 6, 64, 24, 3, 3, (1, 1), (1, 1))),
         ((32, 32, 2), "f16", 1, (2, 6, 5, 128, 40, 3, 3, (2, 1), (1, 0))),
         ((32, 32, 2), "f16", 0, (1, 7, 7, 24, 16, 3, 3, (1, 2), (1, 2))),
         ((32, 64, 2), "bf16", 1, (1, 9, 8, 72, 72, 1, 5, (1, 1), (0, 2)))]


def _conv(case, dt, krsc):
    N, H, W, C, K, R, S, stride, pad = case
    x = wl.small_ints((N, H, W, C), dt, 9500 + C)
    w = wl.small_ints((R, S, C, K), dt, 9600 + K)
    ref = oracle.conv2d(wl.bits(x), wl.bits(w), ODT[dt], stride, pad)
    bias = torch.arange(K, dtype=torch.float32) % 5 - 2
    ref = oracle.epilogue(ref.reshape(-1, K), 0.5, bias.double().numpy(), 1).reshape(ref.shape)
    return x, w.permute(3, 0, 1, 2).contiguous() if krsc else w, bias, ref


@pytest.mark.parametrize("tile,dt,krsc,case", CONVS)
def test_convolution_kernels_on_the_cpu_model(tile, dt, krsc, case):
    x, w, bias, ref = _conv(case, dt, krsc)
    y = torch.full(ref.shape, float("nan"))
    errs = emu.call(al.alcop_conv2d_igemm_fused, x, w, y, case[7], case[8], 0.5, bias, 1, bool(krsc), _sched(tile),
                    reads=[x, w, bias], writes=[y], policy=(1, 1))
    assert not errs, errs[:4]
    assert np.array_equal(y.double().numpy(), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("tile", [(16, 16, 2), (16, 32, 2), (32, 32, 2), (32, 64, 2)])
def test_matrix_kernels_on_the_gpu(tile, tA, tB, dt):
    for (M, N, K) in SHAPES + [(130, 264, 2056)]:
        M, A, B, ref = _problem(M, N, K, dt, tA, tB, 3 if M == 17 else 1)
        for out in (dt, "f32"):
            C = torch.full(ref.shape, float("nan"), dtype=TDT[out], device="cuda")
            (al.alcop_bmm if C.dim() == 3 else al.alcop_gemm)(A.cuda(), B.cuda(), C, _sched(tile), bool(tB),
                                                              transA=bool(tA))
            torch.cuda.synchronize()
            want = torch.from_numpy(ref).to(TDT[out]).double().numpy()
            assert np.array_equal(C.cpu().double().numpy(), want), (M, N, K, out)


@pytest.mark.gpu
@pytest.mark.parametrize("tile,dt,krsc,case", CONVS + [((16, 32, 2), "bf16", 0, (3, 7, 9, 320, 64, 5, 5, (2, 2), (2, 2))),
                                                       ((16, 16, 2), "bf16", 1, (1, 7, 9, 40, 48, 3, 3, (1, 1), (1, 1)))])
def test_convolution_kernels_on_the_gpu(tile, dt, krsc, case):
    x, w, bias, ref = _conv(case, dt, krsc)
    y = torch.full(ref.shape, float("nan"), device="cuda")
    al.alcop_conv2d_igemm_fused(x.cuda(), w.cuda(), y, case[7], case[8], 0.5, bias.cuda(), 1, bool(krsc), _sched(tile))
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().double().numpy(), ref)
