"""Products of operands that are not made of aligned chunks, in one launch (csrc/alcop_direct.hip.h): every
layout at the edges of tiles and k-tiles, exactly.  Around the operands lie infinities, around C NaN."""
import ctypes

import numpy as np
import pytest
import torch

import emu_util as emu
import oracle
import paper_2210_16691_amd as al
import workloads as wl
from test_emulated_unaligned import _embed, _untouched

TDT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
ODT = {"f16": oracle.F16, "bf16": oracle.BF16}
ADT = {"f16": al.F16, "bf16": al.BF16, "f32": al.F32}

# the smallest rows; edges of 64 in every extent; one, two, three and more k-tiles, whole and not
SIZES = [(9, 8, 8), (8, 9, 9), (64, 67, 64), (65, 63, 65), (130, 71, 129), (67, 129, 191), (66, 70, 320), (65, 9, 385)]


def _case(dt, out, size, tA, tB, dev):
    M, N, K = size
    A0 = wl.small_ints((K, M) if tA else (M, K), dt, 50 + M)
    B0 = wl.small_ints((N, K) if tB else (K, N), dt, 60 + N)
    ref = oracle.gemm(wl.bits(A0), wl.bits(B0), ODT[dt], bool(tA), bool(tB))
    bias0 = (torch.arange(N) % 5 - 2).float()
    ref = oracle.epilogue(ref, 0.5, bias0.double().numpy(), 1)
    ref = torch.from_numpy(ref).to(TDT[out]).double().numpy()      # sums here are exact in fp32

    def place(t, offset, pad, fill):
        view, buf = _embed(t, offset, pad, fill=fill)
        moved = buf.to(dev)
        return moved[offset:].as_strided(view.shape, view.stride()), moved

    A, _ = place(A0, 1, 3, float("inf"))
    B, _ = place(B0, 3, 1, float("inf"))
    C, Cbuf = place(torch.full((M, N), float("nan"), dtype=TDT[out]), 1, 2, float("nan"))
    bias = torch.cat([torch.full((1,), float("inf")), bias0]).to(dev)[1:]
    ws = torch.full((al.alcop_unaligned_workspace_bytes(1, M, N, K, ADT[out]),), 255, dtype=torch.uint8, device=dev)
    return A, B, C, Cbuf, bias, ws, ref


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dt,out", [("f16", "f16"), ("bf16", "f32"), ("bf16", "bf16")])
def test_on_the_cpu_model(dt, out, tA, tB):
    for n, size in enumerate(SIZES):
        A, B, C, Cbuf, bias, ws, ref = _case(dt, out, size, tA, tB, "cpu")
        # the workspace is out of bounds: nothing may be copied there
        errs = emu.call(al.alcop_bmm_unaligned, A, B, C, ws, 0.5, bias, 1, transA=bool(tA), transB=bool(tB),
                        reads=[A, B, bias], writes=[C], policy=emu.POLICIES[n % 4])
        assert not errs, (size, errs[:3])
        assert np.array_equal(C.double().numpy(), ref), size
        assert _untouched(Cbuf, C), size


@pytest.mark.parametrize("size,tA,tB", [((9, 5, 8), 0, 0), ((9, 9, 7), 0, 1), ((7, 9, 9), 1, 0), ((30, 30, 2500), 0, 0)])
def test_rows_below_a_chunk_and_long_reductions_are_copied(size, tA, tB):
    A, B, C, Cbuf, bias, ws, ref = _case("f16", "f32", size, tA, tB, "cpu")
    errs = emu.call(al.alcop_bmm_unaligned, A, B, C, ws, 0.5, bias, 1, transA=bool(tA), transB=bool(tB),
                    reads=[A, B, bias], writes=[C, ws])
    assert not errs, errs[:3]
    assert np.array_equal(C.double().numpy(), ref) and _untouched(Cbuf, C)
    assert not bool((ws == 255).all())


@pytest.mark.gpu
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dt,out", [("f16", "f16"), ("bf16", "f32"), ("bf16", "bf16")])
def test_on_the_gpu(dt, out, tA, tB):
    for size in SIZES + [(1021, 333, 257), (300, 2051, 67)]:
        A, B, C, Cbuf, bias, ws, ref = _case(dt, out, size, tA, tB, "cuda:0")
        al.alcop_bmm_unaligned(A, B, C, ws, 0.5, bias, 1, transA=bool(tA), transB=bool(tB))
        torch.cuda.synchronize()
        assert np.array_equal(C.double().cpu().numpy(), ref), size
        assert _untouched(Cbuf, C) and bool((ws == 255).all()), size


def _below_a_chunk(tA, tB):
    """Rows of A, or of B stored N x K, may be fewer than a chunk has elements."""
    return ([(1, 9, 70), (5, 130, 8)] if not tA else []) + ([(9, 1, 70), (130, 5, 8)] if tB else []) + \
           ([(1, 1, 8), (3, 7, 300)] if tB and not tA else [])


def _aligned_result(dt, out, size, tA, tB, alpha, dev):
    """Whole aligned chunks of C, without a bias; A at any element."""
    M, N, K = size
    A0 = wl.small_ints((K, M) if tA else (M, K), dt, 52 + M)
    B = wl.small_ints((N, K) if tB else (K, N), dt, 62 + N).to(dev)
    ref = oracle.epilogue(oracle.gemm(wl.bits(A0), wl.bits(B.cpu()), ODT[dt], bool(tA), bool(tB)), alpha, None, 0)
    buf = torch.full((A0.numel() + 16,), float("inf"), dtype=A0.dtype).to(dev)
    A = buf[1:A0.numel() + 1].view(A0.shape)
    A.copy_(A0)
    Cbuf = torch.full((M + 2, N), float("nan"), dtype=TDT[out]).to(dev)
    ws = torch.full((al.alcop_unaligned_workspace_bytes(1, M, N, K, ADT[out]),), 255, dtype=torch.uint8, device=dev)
    return A, B, Cbuf, Cbuf[1:M + 1], ws, torch.from_numpy(ref).to(TDT[out]).double().numpy()


WHOLE = [(65, 72, 67), (9, 8, 9), (130, 136, 200), (64, 64, 330)]


def _edges(dt, out, tA, tB, dev, call):
    for size in _below_a_chunk(tA, tB):
        A, B, C, Cbuf, bias, ws, ref = _case(dt, out, size, tA, tB, dev)
        call(A, B, C, ws, 0.5, bias, 1)
        assert np.array_equal(C.double().cpu().numpy(), ref), size
        assert _untouched(Cbuf, C) and bool((ws == 255).all()), size
    for n, size in enumerate(WHOLE):
        A, B, Cbuf, C, ws, ref = _aligned_result(dt, out, size, tA, tB, (1.0, 0.5)[n & 1], dev)
        call(A, B, C, ws, (1.0, 0.5)[n & 1], None, 0)
        assert np.array_equal(C.double().cpu().numpy(), ref), size
        assert bool(torch.isnan(Cbuf[[0, -1]]).all()) and bool((ws == 255).all()), size


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dt,out", [("f16", "f16"), ("bf16", "f32")])
def test_small_extents_and_aligned_results_on_the_cpu_model(dt, out, tA, tB):
    def call(A, B, C, ws, alpha, bias, act):
        errs = emu.call(al.alcop_bmm_unaligned, A, B, C, ws, alpha, bias, act, transA=bool(tA), transB=bool(tB),
                        reads=[A, B] + ([] if bias is None else [bias]), writes=[C])
        assert not errs, errs[:3]
    _edges(dt, out, tA, tB, "cpu", call)


@pytest.mark.gpu
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dt,out", [("f16", "f16"), ("bf16", "f32")])
def test_small_extents_and_aligned_results_on_the_gpu(dt, out, tA, tB):
    _edges(dt, out, tA, tB, "cuda:0", lambda A, B, C, ws, alpha, bias, act: al.alcop_bmm_unaligned(
        A, B, C, ws, alpha, bias, act, transA=bool(tA), transB=bool(tB)))


def _both_routes(dt, size, tA, tB, dev, call, auto):
    """The product without copies and with them, each with its relative error against 64 bits, and whether the
    kernel of the copies' route splits K among its waves (fp32 results)."""
    M, N, K = size
    A0, B0 = wl.uniform((K, M) if tA else (M, K), dt, 70 + M), wl.uniform((N, K) if tB else (K, N), dt, 80 + N)
    ref = (A0.double().T if tA else A0.double()) @ (B0.double().T if tB else B0.double())
    A, B = _embed(A0, 1, 0)[1].to(dev)[1:].view(A0.shape), _embed(B0, 1, 0)[1].to(dev)[1:].view(B0.shape)
    ws = torch.empty(al.alcop_unaligned_workspace_bytes(1, M, N, K, al.F32), dtype=torch.uint8, device=dev)
    up = lambda n: (n + 7) // 8 * 8
    padded = auto(al.problem(al.OP_GEMM, up(M) if tA else M, up(N), up(K), ADT[dt], al.F32, transB=bool(tB),
                             transA=bool(tA)))
    out = []
    for sched in (None, padded):
        C = torch.empty(M, N, dtype=torch.float32, device=dev)
        ws.fill_(255)
        call(al.alcop_bmm_unaligned, A, B, C, ws, sched=sched, transA=bool(tA), transB=bool(tB))
        C = C.cpu()
        assert bool((ws == 255).all()) == (sched is None), size        # the route
        out.append((C, ((C.double() - ref).norm() / ref.norm()).item()))
    return out[0], out[1], padded.variant == 3


def _no_more_error(dt, sizes, tA, tB, dev, call, auto):
    split = 0
    for size in sizes:
        (C, direct), (D, copies), splits = _both_routes(dt, size, tA, tB, dev, call, auto)
        if splits:
            split += 1                        # other orders of the sum: the errors' norms differ a little
            assert direct <= 1.05 * copies, (size, direct, copies)
        else:
            assert torch.equal(C, D), size    # the same order
    return split


# most of these get a kernel that splits K among four or eight waves, where copied; all get the direct kernel
ROUTES = [(142, 181, 229), (201, 99, 401), (260, 131, 395), (330, 300, 501), (67, 66, 65), (90, 75, 121), (435, 386, 385)]


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_no_more_error_than_with_copies_on_the_cpu_model(tA, tB):
    def call(f, A, B, C, ws, **kw):
        errs = emu.call(f, A, B, C, ws, reads=[A, B], writes=[C, ws], **kw)
        assert not errs, errs[:3]

    def auto(prob):
        with emu._swapped():
            return al.alcop_sched_auto(prob)
    split = _no_more_error("f16", ROUTES, tA, tB, "cpu", call, auto)
    assert split >= (0 if tA and not tB else 4)      # the model holds no such kernel for this layout


def test_a_pick_read_from_a_file_takes_the_same_route(tmp_path):
    A, B, C, Cbuf, bias, ws, ref = _case("f16", "f32", (150, 181, 229), 0, 0, "cpu")
    for step in ("picked", "read"):            # the entry that is read replaces the one that was picked
        assert not emu.call(al.alcop_bmm_unaligned, A, B, C, ws, 0.5, bias, 1, reads=[A, B, bias], writes=[C, ws])
        assert bool((ws == 255).all()), step
        with emu._swapped():
            assert al.alcop_cache_save(str(tmp_path / "picks")) >= 1
            assert al.alcop_cache_load(str(tmp_path / "picks")) >= 1


@pytest.mark.gpu
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dt", ["f16", "bf16"])
def test_no_more_error_than_with_copies_on_the_gpu(dt, tA, tB):
    assert _no_more_error(dt, ROUTES, tA, tB, "cuda:0", lambda f, *a, **kw: f(*a, **kw), al.alcop_sched_auto) >= 4


def test_init_loads_the_kernels_of_unaligned_calls():
    L = emu.lib()
    assert L.alcop_init() == al.OK
    assert L.emu_loaded() == 40 + 2             # two types, four layouts, two depths, and three of partial sums; the copies


@pytest.mark.gpu
def test_captured_after_alcop_init():
    al.alcop_init()
    small, odd = (142, 181, 229), (1021, 1531, 767)           # without copies, with them
    make = lambda size, seed: (wl.uniform(size[::2], "bf16", seed).to("cuda:0"), wl.uniform(size[:0:-1], "bf16", seed + 1).to("cuda:0"))
    ops = [make(small, 90), make(odd, 92)]
    outs = [torch.empty(M, N, dtype=torch.bfloat16, device="cuda:0") for M, N, _ in (small, odd)]
    ws = [torch.empty(al.alcop_unaligned_workspace_bytes(1, *s, al.BF16), dtype=torch.uint8, device="cuda:0")
          for s in (small, odd)]
    x, w = wl.uniform((2, 30, 31, 3), "bf16", 94).to("cuda:0"), wl.uniform((3, 3, 3, 21), "bf16", 95).to("cuda:0")
    outs.append(torch.empty(2, 30, 31, 21, dtype=torch.bfloat16, device="cuda:0"))
    ws.append(torch.empty(al.alcop_conv2d_unaligned_workspace_bytes(2, 30, 31, 3, 21, 3, 3, (1, 1), (1, 1), (1, 1), al.BF16),
                          dtype=torch.uint8, device="cuda:0"))

    def work(stream):
        for (A, B), C, s in zip(ops, outs, ws):
            al.alcop_bmm_unaligned(A, B, C, s, stream=stream)
        al.alcop_conv2d_igemm_unaligned(x, w, outs[2], ws[2], (1, 1), (1, 1), stream=stream)

    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            work(torch.cuda.current_stream())
    torch.cuda.synchronize()
    for rep in range(4):
        for (A, B), size in zip(ops, (small, odd)):
            for t, new in zip((A, B), make(size, 100 + rep)):
                t.copy_(new)
        x.copy_(wl.uniform((2, 30, 31, 3), "bf16", 110 + rep).to("cuda:0"))
        work(torch.cuda.current_stream())
        torch.cuda.synchronize()
        want = [C.clone() for C in outs]
        for C in outs:
            C.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for C, ref in zip(outs, want):
            assert torch.equal(C.view(torch.int16), ref.view(torch.int16)), rep


@pytest.mark.parametrize("size,tA,tB", [((8, 7800001, 129), 0, 0), ((8, 7800001, 129), 1, 0), ((3000001, 20, 321), 1, 0)])
def test_a_product_that_its_kernel_refuses_stays_refused(size, tA, tB):
    # padded, K rounded up to whole k-tiles reaches 2^31 bytes: refused before anything is launched,
    # also where the product without copies looks cheaper (addresses that nothing may touch)
    M, N, K = size
    A, B, C, ws = (ctypes.c_void_p(i << 40) for i in (1, 2, 3, 4))
    L = emu.lib()
    L.emu_reset(1, 0)
    need = L.alcop_unaligned_workspace_bytes(1, M, N, K, al.F16)
    assert need > 0
    rc = L.alcop_bmm_unaligned(A, B, C, 1, M, N, K, M if tA else K, K if tB else N, N, 0, 0, 0, tA, tB, al.F16, al.F16,
                               None, None, ws, need, None)
    assert rc == al.ERR_SIZE and L.emu_error_count() == 0
