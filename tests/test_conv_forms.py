"""Convolutions with few channels, which are laid out for the gather with several pixels (pair form)
or a whole filter row (window form) per 16-byte chunk, and outputs whose rows are not made of such
chunks: exact on small integers, in the CPU model of the hardware (bounds checks) and on the GPU."""
import numpy as np
import pytest
import torch

import emu_util as emu
import oracle
import paper_2210_16691_amd as al
import workloads as wl

# (N, H, W, C, K, R, S, stride, pad): pair form with px = 2, 4 and 8 pixels a chunk, left padding of
# every parity and none, the last window ending inside, at and past the image; window form for odd
# strides, one-element windows and windows wider than the image; a wide and a ragged K
CASES = [(2, 13, 14, 3, 64, 7, 7, (2, 2), (3, 3)), (1, 9, 11, 4, 8, 3, 3, (2, 2), (1, 1)),
         (1, 10, 9, 3, 61, 5, 5, (1, 4), (2, 0)), (2, 6, 17, 2, 16, 3, 5, (2, 4), (1, 2)),
         (1, 7, 33, 1, 24, 3, 7, (1, 8), (1, 3)), (2, 8, 8, 1, 9, 7, 7, (1, 1), (3, 3)),
         (1, 5, 6, 3, 17, 3, 3, (1, 1), (1, 1)), (1, 4, 3, 5, 8, 1, 9, (1, 3), (0, 4)),
         (1, 6, 6, 12, 7, 3, 3, (1, 1), (0, 0))]


def _inputs(case, dt):
    N, H, W, C, K, R, S, stride, pad = case
    x0, w0 = wl.small_ints((N, H, W, C), dt, 9100 + C), wl.small_ints((R, S, C, K), dt, 9200 + K)
    bias = torch.arange(K, dtype=torch.float32) % 7 - 3
    ref = oracle.conv2d(wl.bits(x0), wl.bits(w0), oracle.F16 if dt == "f16" else oracle.BF16, stride, pad)
    ref = oracle.epilogue(ref.reshape(-1, K), 1.0, bias.double().numpy(), 1).reshape(ref.shape)
    return x0, w0, bias, ref


def _embed(t, device="cpu", fill=0.0):
    buf = torch.full((t.numel() + 2,), fill, dtype=t.dtype, device=device)
    v = buf[1:-1].view(t.shape)
    v.copy_(t)
    return v, buf


@pytest.mark.parametrize("case", CASES)
def test_forms_on_the_cpu_model(case):
    N, H, W, C, K, R, S, stride, pad = case
    x0, w0, bias, ref = _inputs(case, "f16")
    x, w = _embed(x0)[0], _embed(w0)[0]
    y, yb = _embed(torch.full(ref.shape, float("nan"), dtype=torch.float16), fill=float("nan"))
    ws = torch.empty(al.alcop_conv2d_unaligned_workspace_bytes(N, H, W, C, K, R, S, stride, pad, (1, 1), al.F16),
                     dtype=torch.uint8)
    errs = emu.call(al.alcop_conv2d_igemm_unaligned, x, w, y, ws, stride, pad, (1, 1), 1.0, bias, 1,
                    reads=[x, w, bias], writes=[y, ws], policy=(1, 0))
    assert not errs, errs[:4]
    assert np.array_equal(y.double().numpy(), ref)
    assert torch.isnan(yb[0]) and torch.isnan(yb[-1])


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("case", CASES + [(3, 57, 61, 3, 64, 7, 7, (2, 2), (3, 3)),
                                          (2, 40, 40, 1, 96, 5, 5, (1, 1), (2, 2))])
def test_forms_on_the_gpu(case, dt):
    N, H, W, C, K, R, S, stride, pad = case
    x0, w0, bias, ref = _inputs(case, dt)
    x, w = _embed(x0, "cuda")[0], _embed(w0, "cuda")[0]
    y, yb = _embed(torch.full(ref.shape, float("nan")), "cuda", float("nan"))
    ws = torch.empty(al.alcop_conv2d_unaligned_workspace_bytes(N, H, W, C, K, R, S, stride, pad, (1, 1), al.F32),
                     dtype=torch.uint8, device="cuda")
    al.alcop_conv2d_igemm_unaligned(x, w, y, ws, stride, pad, (1, 1), 1.0, bias.cuda(), 1)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().double().numpy(), ref)
    assert bool(torch.isnan(yb[0])) and bool(torch.isnan(yb[-1]))


def _finite(x0, w0, stride, pad):
    y = torch.nn.functional.conv2d(x0.double().permute(0, 3, 1, 2), w0.double().permute(3, 2, 0, 1), None, stride, pad)
    return torch.isfinite(y).permute(0, 2, 3, 1)


def _poisoned(case, col, dt="f16"):
    """Inputs with an infinity and a NaN in column `col` (modulo the width) of two rows."""
    N, H, W, C, K, R, S, stride, pad = case
    x0, w0, _, _ = _inputs(case, dt)
    x0[0, H // 2, col % W, C - 1] = float("inf")
    x0[N - 1, 0, (col + 3) % W, 0] = float("nan")
    return x0, w0, _finite(x0, w0, stride, pad)


# further: an even filter, whose windows are whole chunks; a halo too wide for the LDS; a last chunk with
# one pixel of four, three of four and an odd number of elements
RAGGED = [(1, 9, 12, 3, 16, 4, 4, (2, 2), (1, 1)), (1, 7, 2600, 4, 8, 7, 5, (2, 2), (3, 2)),
          (1, 6, 17, 2, 16, 3, 7, (2, 4), (1, 2)), (1, 4, 40, 1, 8, 2, 13, (1, 8), (0, 5))]


@pytest.mark.parametrize("col", [4, 5, 7])
@pytest.mark.parametrize("case", CASES + RAGGED)
def test_non_finite_pixels_reach_their_windows_only(case, col):
    # padding must not multiply a neighbouring pixel by a zero weight (0 * inf)
    N, H, W, C, K, R, S, stride, pad = case
    x, w, want = _poisoned(case, col)
    y = torch.zeros(want.shape, dtype=torch.float32)
    ws = torch.empty(al.alcop_conv2d_unaligned_workspace_bytes(N, H, W, C, K, R, S, stride, pad, (1, 1), al.F32),
                     dtype=torch.uint8)
    errs = emu.call(al.alcop_conv2d_igemm_unaligned, x, w, y, ws, stride, pad, reads=[x, w], writes=[y, ws])
    assert not errs, errs[:4]
    assert torch.equal(torch.isfinite(y), want)


# one and a half tiles of the widest kernel, K not a multiple of a k-tile
STEM = (2, 25, 27, 3, 72, 7, 7, (2, 2), (3, 3))


def _loaded(tmp_path, tile, dt, M):
    """Makes `tile` the schedule of the stem's inner product (224 deep, windows of 32 elements)."""
    f = tmp_path / "cache"
    key = al.sched(tile[0], tile[1], 64, 64, 64, tile[2], 2, 1, 1, 0, 4).key()
    f.write_text("2 1 %d 72 224 0 0 %d 2 32 : %s\n" % (M, dt == "bf16", " ".join(map(str, key))))
    return al.alcop_cache_load(str(f))


@pytest.mark.parametrize("tile", [(256, 64, 3), (128, 128, 2), (128, 64, 3), (64, 64, 2)])
def test_every_tile_clears_what_lies_past_a_window(tile, tmp_path, monkeypatch, capfd):
    N, H, W, C, K, R, S, stride, pad = STEM
    x, w, want = _poisoned(STEM, 5)
    y = torch.zeros(want.shape, dtype=torch.float32)
    ws = torch.empty(al.alcop_conv2d_unaligned_workspace_bytes(N, H, W, C, K, R, S, stride, pad, (1, 1), al.F32),
                     dtype=torch.uint8)
    monkeypatch.setenv("ALCOP_LOG", "1")
    with emu._swapped():
        assert _loaded(tmp_path, tile, "f16", want[..., 0].numel()) == 1
    errs = emu.call(al.alcop_conv2d_igemm_unaligned, x, w, y, ws, stride, pad, reads=[x, w], writes=[y, ws])
    assert "tile %dx%dx64" % tile[:2] in capfd.readouterr().err
    assert not errs, errs[:4]
    assert torch.equal(torch.isfinite(y), want)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("tile", [(256, 64, 2), (256, 64, 3), (128, 128, 2), (128, 128, 3), (128, 64, 2), (128, 64, 3),
                                  (64, 128, 2), (64, 64, 2)])
def test_every_tile_clears_what_lies_past_a_window_on_the_gpu(tile, dt, tmp_path):
    N, H, W, C, K, R, S, stride, pad = STEM
    x0, w0, bias, ref = _inputs(STEM, dt)
    xp, wp, want = _poisoned(STEM, 5, dt)
    ws = torch.empty(al.alcop_conv2d_unaligned_workspace_bytes(N, H, W, C, K, R, S, stride, pad, (1, 1), al.F32),
                     dtype=torch.uint8, device="cuda")
    assert _loaded(tmp_path, tile, dt, want[..., 0].numel()) == 1
    y = torch.zeros(want.shape, device="cuda")
    al.alcop_conv2d_igemm_unaligned(xp.cuda(), wp.cuda(), y, ws, stride, pad)
    z = torch.zeros(want.shape, device="cuda")
    al.alcop_conv2d_igemm_unaligned(x0.cuda(), w0.cuda(), z, ws, stride, pad, (1, 1), 1.0, bias.cuda(), 1)
    torch.cuda.synchronize()
    assert torch.equal(torch.isfinite(y).cpu(), want)
    assert np.array_equal(z.cpu().double().numpy(), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f16", "bf16"])
def test_non_finite_pixels_reach_their_windows_only_on_the_gpu(dt):
    for case in CASES + RAGGED + [(3, 57, 61, 3, 64, 7, 7, (2, 2), (3, 3)), (40, 57, 61, 3, 64, 7, 7, (2, 2), (3, 3)),
                                  (40, 57, 61, 3, 128, 5, 5, (2, 2), (2, 2))]:
        N, H, W, C, K, R, S, stride, pad = case
        ws = torch.empty(al.alcop_conv2d_unaligned_workspace_bytes(N, H, W, C, K, R, S, stride, pad, (1, 1), al.F32),
                         dtype=torch.uint8, device="cuda")
        for col in (4, 5):
            x, w, want = _poisoned(case, col, dt)
            y = torch.zeros(want.shape, device="cuda")
            al.alcop_conv2d_igemm_unaligned(x.cuda(), w.cuda(), y, ws, stride, pad)
            torch.cuda.synchronize()
            assert torch.equal(torch.isfinite(y).cpu(), want), (case, col)
