"""Products whose kernel takes its arguments in one 64-byte line (SmallArgs): every form of a call that is
described so, and the ones next to it that are not (a batch with a bias), against the oracle, exactly."""
import numpy as np
import pytest
import torch

import emu_util as emu
import oracle
import paper_2210_16691_amd as al
import workloads as wl

TDT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
ODT = {"f16": oracle.F16, "bf16": oracle.BF16}
ADT = {"f16": al.F16, "bf16": al.BF16, "f32": al.F32}

# sizes at the edges of 16, 32 and 64 wide tiles; the last has 13 rows of 16-wide tiles (a band of eight and one
# of five) and more than one column of every tile
SIZES = [(1, 8, 8), (17, 40, 72), (65, 72, 200), (200, 72, 72)]
# (transA, transB, batch, bias, relu, alpha)
FORMS = [(0, 0, 1, 1, 1, 0.5), (0, 1, 1, 0, 1, 1.0), (1, 0, 1, 0, 0, 1.0), (1, 1, 1, 0, 0, 1.0), (1, 0, 2, 0, 0, 1.0),
         (0, 0, 3, 0, 0, 0.5), (0, 1, 2, 1, 1, 1.0)]


def _case(dt, out, size, form, dev):
    (M, N, K), (tA, tB, b, bias, relu, alpha) = size, form
    if tA:
        M = (M + 7) // 8 * 8
    A = wl.small_ints((b, K, M) if tA else (b, M, K), dt, 10 + M)
    B = wl.small_ints((b, N, K) if tB else (b, K, N), dt, 20 + N)
    ref = oracle.bmm(wl.bits(A), wl.bits(B), ODT[dt], bool(tA), bool(tB))
    bv = (torch.arange(N) % 5 - 2).float() if bias else None
    ref = oracle.epilogue(ref, alpha, bv.double().numpy() if bias else None, relu)
    ref = torch.from_numpy(ref).to(TDT[out]).double().numpy()      # sums here are exact in fp32
    C = torch.full((b, M, N + 8), float("nan"), dtype=TDT[out], device=dev)[:, :, :N]
    return A.to(dev), B.to(dev), C, bv.to(dev) if bias else None, ref


def _run(call, A, B, C, bias, form):
    tA, tB, b, _, relu, alpha = form
    if tA:                                   # no fused form
        kw = dict(transA=True, transB=bool(tB))
        return call(al.alcop_gemm, A[0], B[0], C[0], **kw) if b == 1 else call(al.alcop_bmm, A, B, C, **kw)
    kw = dict(bias=bias, act=relu, transB=bool(tB))
    if b == 1:
        return call(al.alcop_gemm_fused, A[0], B[0], C[0], alpha, **kw)
    return call(al.alcop_bmm_fused, A, B, C, alpha, **kw)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("dt,out", [("f16", "f16"), ("bf16", "f32"), ("bf16", "bf16")])
def test_on_the_cpu_model(dt, out, form):
    ran, banded = 0, 0
    for n, size in enumerate(SIZES):
        A, B, C, bias, ref = _case(dt, out, size, form, "cpu")
        b, M, N = C.shape
        prob = al.problem(al.OP_BMM if b > 1 else al.OP_GEMM, M, N, size[2], ADT[dt], ADT[out],
                          transB=bool(form[1]), transA=bool(form[0]), batch=b)
        small = [s for s in emu.space(prob, opt_in=True) if s.variant == 3 or (s.variant == 0 and s.bm == s.bn == 64)]
        for s in small:
            C.fill_(float("nan"))
            errs = _run(lambda f, *a, **k: emu.call(f, *a, sched=s, reads=[A, B] + ([bias] if bias is not None else []),
                                                    writes=[C], policy=emu.POLICIES[n], **k), A, B, C, bias, form)
            assert not errs, (s, errs[:3])
            assert np.array_equal(C.double().numpy(), ref), (s, size)
            ran += 1
            banded += s.bm == 16 and s.raster == 1 and M > 8 * 16
    assert ran and (banded or dt != "f16" or form[0])      # the model holds 16-wide tiles for these


@pytest.mark.gpu
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("dt,out", [("f16", "f16"), ("bf16", "f32"), ("bf16", "bf16")])
def test_on_the_gpu(dt, out, form):
    for size in SIZES + [(256, 256, 256), (16, 3072, 768)]:
        A, B, C, bias, ref = _case(dt, out, size, form, "cuda:0")
        _run(lambda f, *a, **k: f(*a, **k), A, B, C, bias, form)
        torch.cuda.synchronize()
        assert np.array_equal(C.double().cpu().numpy(), ref), size


def _schedules(dt, out, size, form):
    """The kernels of a product that take these arguments: waves that split K, 64 x 64 tiles."""
    tA, tB, b = form[:3]
    M = (size[0] + 7) // 8 * 8 if tA else size[0]
    prob = al.problem(al.OP_BMM if b > 1 else al.OP_GEMM, M, size[1], size[2], ADT[dt], ADT[out], transB=bool(tB),
                      transA=bool(tA), batch=b)
    tiles = [(16, 16, 2, 1, 0, 3), (16, 32, 2, 1, 0, 3), (32, 32, 2, 1, 0, 3), (32, 64, 2, 1, 0, 3)]
    found = [al.sched(bm, bn, 64, bm, bn, st, r, f, 1, 0, v) for bm, bn, st, r, f, v in tiles]
    found += [al.sched(64, 64, 64, 32, 32, 3, 2, 1), al.sched(64, 64, 64, 32, 32, 4, 2, 1), al.sched(64, 64, 32, 32, 32, 3, 1, 0)]
    return [s for s in found if al.alcop_sched_supported(prob, s) == al.OK]


@pytest.mark.gpu
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("dt,out", [("f16", "f16"), ("bf16", "f32"), ("bf16", "bf16")])
def test_every_kernel_on_the_gpu(dt, out, form):
    for size in SIZES + [(520, 136, 264)]:
        A, B, C, bias, ref = _case(dt, out, size, form, "cuda:0")
        scheds = _schedules(dt, out, size, form)
        assert len(scheds) >= 4, (size, scheds)
        for s in scheds:
            C.fill_(float("nan"))
            _run(lambda f, *a, **k: f(*a, sched=s, **k), A, B, C, bias, form)
            torch.cuda.synchronize()
            assert np.array_equal(C.double().cpu().numpy(), ref), (s, size)
