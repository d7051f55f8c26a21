"""The C++ argument marshalling of the hot entry points: leaves to the Python code what it does not
take, and otherwise makes the same call (same bits) as the ctypes path."""
import ctypes

import pytest
import torch

import paper_2210_16691_amd as al


def test_arguments_it_does_not_take_are_left_to_python():
    al.lib()
    h = lambda *s: torch.zeros(*s, dtype=torch.float16)
    # host tensors, whatever their shapes
    assert al._marshal.mm(h(8, 16), h(16, 8), h(8, 8), False, False, None, None) is None
    assert al._marshal.conv(h(1, 4, 4, 8), h(3, 3, 8, 8), h(1, 2, 2, 8), (1, 1), (0, 0), (1, 1), False, None, None,
                            1.0, None, 0) is None
    assert al._marshal.mm(None, h(16, 8), h(8, 8), False, False, None, None) is None
    with pytest.raises(ValueError):
        al.alcop_gemm(h(8, 16), h(8, 8), h(8, 8))


def _mm(f, tB=False, tA=False, b=0, pitch=0, **kw):
    g = torch.Generator().manual_seed(7)
    sh = lambda r, c: ((b, r, c + pitch) if b else (r, c + pitch))
    mk = lambda r, c: torch.rand(sh(r, c), generator=g).half().cuda()[..., :c]
    M, N, K = 72, 64, 96
    A, B = mk(*((K, M) if tA else (M, K))), mk(*((N, K) if tB else (K, N)))
    return lambda C: f(A, B, C, **dict(kw, **({"transB": tB} if tB else {}), **({"transA": tA} if tA else {})))


class _Recorder:
    """The marshalling module, with the results of its calls written down."""

    def __init__(self, module):
        self.module, self.results = module, []

    def __getattr__(self, name):
        def f(*args):
            self.results.append(getattr(self.module, name)(*args))
            return self.results[-1]
        return f


@pytest.mark.gpu
@pytest.mark.parametrize("case", ["gemm", "gemm_ta", "fused", "bmm", "bmm_fused", "any", "conv", "krsc", "fusedconv",
                                  "dilated", "convany"])
def test_same_bits_as_the_ctypes_path(case):
    bias = torch.linspace(-1, 1, 64).cuda()
    s = al.sched(64, 64, 64, 32, 32, 3, 2, 1)
    side = torch.cuda.Stream()
    x, w = torch.rand(2, 9, 9, 64).half().cuda(), torch.rand(3, 3, 64, 64).half().cuda()
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    shape = (3, 72, 64) if case in ("bmm", "bmm_fused") else (2, 7, 7, 64) if "conv" in case or case == "krsc" else (72, 64)
    if case == "dilated":
        shape = (2, 5, 5, 64)
    run = {"gemm": _mm(al.alcop_gemm, sched=s), "gemm_ta": _mm(al.alcop_gemm, tA=True, stream=side),
           "fused": _mm(al.alcop_gemm_fused, tB=True, alpha=0.5, bias=bias, act=1, pitch=8),
           "bmm": _mm(al.alcop_bmm, b=3), "bmm_fused": _mm(al.alcop_bmm_fused, b=3, tB=True, alpha=2, bias=bias),
           "any": _mm(lambda A, B, C, **k: al.alcop_bmm_unaligned(A, B, C, ws, 0.5, bias, 1, **k), pitch=3),
           "conv": lambda y: al.alcop_conv2d_igemm(x, w, y),
           "krsc": lambda y: al.alcop_conv2d_igemm_krsc(x, w.permute(3, 0, 1, 2).contiguous(), y, sched=None),
           "fusedconv": lambda y: al.alcop_conv2d_igemm_fused(x, w, y, alpha=0.25, bias=bias, act=1),
           "dilated": lambda y: al.alcop_conv2d_igemm_dilated(x, w, y, dilation=(2, 2), bias=bias),
           "convany": lambda y: al.alcop_conv2d_igemm_unaligned(x, w, y, ws, bias=bias)}[case]
    al.lib()
    outs = []
    for native in (al._lib, None):
        module, keep = al._marshal, al._marshal_lib
        al._marshal, al._marshal_lib = _Recorder(module), native
        try:
            C = torch.full(shape, float("nan"), dtype=torch.float16, device="cuda")
            torch.cuda.synchronize()
            run(C)
            torch.cuda.synchronize()
            assert al._marshal.results == ([0] if native else [])   # it took the call, or was not asked
        finally:
            al._marshal, al._marshal_lib = module, keep
        outs.append(C)
    assert not torch.isnan(outs[0]).any()
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))


@pytest.mark.gpu
def test_arguments_of_other_types_stay_refused():
    # 44 bytes of something else have the size of a schedule
    s = al.sched(64, 64, 64, 32, 32, 3, 2, 1)
    A = torch.zeros(64, 64, dtype=torch.float16, device="cuda")
    for other in (bytes(s), bytearray(s), torch.tensor(s.key(), dtype=torch.int32).numpy()):
        with pytest.raises(TypeError):
            al.alcop_gemm(A, A, torch.empty_like(A), sched=other)
    with pytest.raises(TypeError):
        al.alcop_gemm(A, A, torch.empty_like(A), transB=None)
    al.alcop_gemm(A, A, torch.empty_like(A), sched=s)
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_an_exception_out_of_the_library_is_raised_under_the_interpreter_lock():
    # the C++ runtime's own thrower in the place of the entry points: nothing is launched
    al.lib()
    addr = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    L = al._lib
    A = torch.zeros(64, 64, dtype=torch.float16, device="cuda")
    try:
        al._marshal.init(al.Sched, *[addr(ctypes.CDLL("libstdc++.so.6")._ZSt17__throw_bad_allocv)] * 5)
        for _ in range(3):
            with pytest.raises(RuntimeError):
                al.alcop_gemm(A, A, torch.empty_like(A))
    finally:
        al._marshal.init(al.Sched, *[addr(f) for f in (L.alcop_gemm_fused, L.alcop_bmm_fused, L.alcop_bmm_unaligned,
                                                       L.alcop_conv2d_igemm_dilated, L.alcop_conv2d_igemm_unaligned)])
    al.alcop_gemm(A, A, torch.empty_like(A))
    torch.cuda.synchronize()
