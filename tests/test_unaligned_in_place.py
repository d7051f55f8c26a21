"""The unaligned entry points read operands that need no padding where they lie.  What a copy of
every operand used to guarantee must still hold, here on the CPU model of the hardware: the result
may lie on an operand."""
import numpy as np
import pytest
import torch

import emu_util as emu
import oracle
import paper_2210_16691_amd as al
import workloads as wl


def _odd(t):
    """A copy of t at an address that is a multiple of its element size only."""
    v = torch.zeros(t.numel() + 1, dtype=t.dtype)[1:].view(t.shape)
    return v.copy_(t)


def _aligned(*shape, dtype=torch.float16):
    n = int(np.prod(shape))
    buf = torch.zeros(n + 64, dtype=dtype)
    off = (-buf.data_ptr() % 64) // buf.element_size()
    return buf[off:off + n].view(*shape)


def _mm(A, B, C, **kw):
    M, K = A.shape[-2:][::-1] if kw.get("transA") else A.shape[-2:]
    code = {torch.float16: al.F16, torch.float32: al.F32}[C.dtype]
    ws = torch.empty(al.alcop_unaligned_workspace_bytes(A.shape[0] if A.dim() == 3 else 1, M, C.shape[-1], K, code),
                     dtype=torch.uint8)
    bias = kw.get("bias")
    return emu.call(al.alcop_bmm_unaligned, A, B, C, ws, reads=[A, B] + ([] if bias is None else [bias]),
                    writes=[C, ws], **kw)


def _ref(A, B, tA=False, tB=False):
    return oracle.gemm(wl.bits(A.contiguous()), wl.bits(B.contiguous()), oracle.F16, tA, tB)


@pytest.mark.parametrize("on", ["A", "B", "A_shifted", "A_transposed"])
def test_a_product_may_overwrite_its_operand(on):
    M, N, K = (130, 200, 200) if on[0] == "A" else (200, 136, 200)
    if on == "A_transposed":
        M = N = K = 200
    A0, B0 = wl.small_ints((M, K), "f16", 31), wl.small_ints((K, N), "f16", 32)
    ref = _ref(A0, B0, on == "A_transposed")
    mem = _aligned(250, 200)
    if on[0] == "A":
        A, B = mem[:M], _odd(B0)
        A.copy_(A0)
        C = mem[40:40 + M] if on == "A_shifted" else mem[:M]
    else:
        A, B = _odd(A0), mem.view(-1)[:K * N].view(K, N)
        B.copy_(B0)
        C = mem.view(-1)[:M * N].view(M, N)
    errs = _mm(A, B, C, transA=on == "A_transposed")
    assert not errs, errs[:4]
    assert np.array_equal(C.double().numpy(), ref)


def test_a_batched_product_may_overwrite_another_entry():
    b, M, N, K = 3, 72, 64, 64
    A0, B0 = wl.small_ints((b, M, K), "f16", 33), wl.small_ints((b, K, N), "f16", 34)
    mem = _aligned(b + 1, M, K)
    A, C = mem[:b], mem[1:]                 # entry i of C on entry i + 1 of A
    A.copy_(A0)
    errs = _mm(A, _odd(B0), C)
    assert not errs, errs[:4]
    for i in range(b):
        assert np.array_equal(C[i].double().numpy(), _ref(A0[i], B0[i])), i


def test_a_product_may_overwrite_its_bias():
    M, N, K = 200, 64, 24
    A0, B0 = wl.small_ints((M, K), "f16", 35), wl.small_ints((K, N), "f16", 36)
    C = _aligned(M, N, dtype=torch.float32)
    bias = C[0]
    bias.copy_(torch.arange(N) % 9 - 4)
    ref = oracle.epilogue(_ref(A0, B0), 1.0, bias.double().numpy(), 0)
    errs = _mm(_odd(A0), B0, C, bias=bias)
    assert not errs, errs[:4]
    assert np.array_equal(C.double().numpy(), ref)


@pytest.mark.parametrize("on", ["x", "w", "bias"])
def test_a_convolution_may_overwrite_its_operand(on):
    N, H, W, C, K = 1, 20, 18, 16, 16
    x0, w0 = wl.small_ints((N, H, W, C), "f16", 37), wl.small_ints((3, 3, C, K), "f16", 38)
    ref = oracle.conv2d(wl.bits(x0), wl.bits(w0), oracle.F16, (1, 1), (1, 1))
    b0 = torch.arange(K, dtype=torch.float32) % 7 - 3
    ref = oracle.epilogue(ref.reshape(-1, K), 1.0, b0.double().numpy(), 0).reshape(ref.shape)
    y = _aligned(N, H, W, K, dtype=torch.float32 if on == "bias" else torch.float16)
    flat = y.view(-1)
    x, w, bias = _odd(x0), _odd(w0), b0.clone()
    if on == "x":
        x = flat.view(x0.shape).copy_(x0)
    elif on == "w":
        w = flat[:w0.numel()].view(w0.shape).copy_(w0)
    else:
        bias = flat[:K].copy_(b0)
    ws = torch.empty(al.alcop_conv2d_unaligned_workspace_bytes(N, H, W, C, K, 3, 3, (1, 1), (1, 1), (1, 1), al.F32),
                     dtype=torch.uint8)
    errs = emu.call(al.alcop_conv2d_igemm_unaligned, x, w, y, ws, (1, 1), (1, 1), bias=bias,
                    reads=[x, w, bias], writes=[y, ws])
    assert not errs, errs[:4]
    assert np.array_equal(y.double().numpy(), ref)


def test_an_operand_whose_rounded_span_is_too_long_is_copied():
    # the loaders address K rounded up to a k-tile of rows: 64 rows at this pitch are 4 GiB
    M, N, K, pitch = 5, 8, 8, 1 << 25
    A0, B0 = wl.small_ints((M, K), "f16", 41), wl.small_ints((K, N), "f16", 42)
    buf = torch.empty(K * pitch + 8, dtype=torch.float16)
    B = buf[-buf.data_ptr() // 2 % 8:].as_strided((K, N), (pitch, 1)).copy_(B0)
    A, C = _aligned(M, K).copy_(A0), _odd(torch.full((M, N), float("nan"), dtype=torch.float16))
    assert B.data_ptr() % 16 == 0
    errs = _mm(A, B, C)
    assert not errs, errs[:4]
    assert np.array_equal(C.double().numpy(), _ref(A0, B0))
    At = buf[-buf.data_ptr() // 2 % 8:].as_strided((K, 8), (pitch, 1)).copy_(B0)       # A stored K x M
    D = _odd(torch.full((8, N), float("nan"), dtype=torch.float16))
    errs = _mm(At, _aligned(K, N).copy_(B0), D, transA=True)
    assert not errs, errs[:4]
    assert np.array_equal(D.double().numpy(), _ref(B0, B0, True))


def _far_rows(device, kind):
    """Three rows of C 2^30 + 1 elements apart (2^30 + 8 for the aligned form)."""
    M, N, K, pitch = 3, 24, 40, (1 << 30) + (8 if kind == "aligned" else 1)
    A0, B0 = wl.small_ints((M, K), "f16", 43), wl.small_ints((K, N), "f16", 44)
    buf = torch.empty(2 * pitch + N + 8, dtype=torch.float16, device=device)
    C = buf[-buf.data_ptr() // 2 % 8:].as_strided((M, N), (pitch, 1))
    C.fill_(float("nan"))
    return A0, B0, C


@pytest.mark.parametrize("kind", ["aligned", "odd", "waves_split_k"])
def test_rows_of_the_result_may_be_far_apart(kind):
    A0, B0, C = _far_rows("cpu", kind)
    s = al.sched(64, 64, 64, 32, 32, 3, 2, 1) if kind != "waves_split_k" else al.sched(16, 16, 64, 16, 16, 2, 1, 0, variant=3)
    errs = _mm(_odd(A0), B0, C, sched=s)
    assert not errs, errs[:4]
    assert np.array_equal(C.double().numpy(), _ref(A0, B0))
    with pytest.raises(al.AlcopError) as e:            # the other entry points keep their limit
        emu.call(al.alcop_gemm, A0, B0, C, reads=[A0, B0], writes=[C])
    assert e.value.code in (al.ERR_SIZE, al.ERR_ALIGN)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["aligned", "odd", "persistent", "waves_split_k"])
def test_rows_of_the_result_may_be_far_apart_on_the_gpu(kind):
    A0, B0, C = _far_rows("cuda", kind)
    s = {"persistent": al.sched(64, 64, 64, 32, 32, 3, 2, 1, variant=2),
         "waves_split_k": al.sched(16, 16, 64, 16, 16, 2, 1, 0, variant=3)}.get(kind, al.sched(64, 64, 64, 32, 32, 3, 2, 1))
    ws = torch.empty(al.alcop_unaligned_workspace_bytes(1, 3, 24, 40, al.F16), dtype=torch.uint8, device="cuda")
    al.alcop_bmm_unaligned(A0.cuda(), B0.cuda(), C, ws, sched=s)
    torch.cuda.synchronize()
    assert np.array_equal(C.cpu().double().numpy(), _ref(A0, B0))
