"""Convolution kernels with a resident patch for any geometry (schedule variant 4): exact on small
integers where a patch can go wrong (rows and images that end inside a tile, strides, dilation,
channel counts that 64 does not divide, padding wider than the filter), in the CPU model of the
hardware and on the GPU."""
import numpy as np
import pytest
import torch

import emu_util as emu
import oracle
import paper_2210_16691_amd as al
import workloads as wl

TDT = {"f16": torch.float16, "bf16": torch.bfloat16}
ODT = {"f16": oracle.F16, "bf16": oracle.BF16}


def _sched(t):
    return al.sched(t[0], t[1], 64, 64, 64, t[2], 2, 1, 1, 0, 4)


# N, H, W, C, K, R, S, stride, pad, dilation
GEOM = [(2, 9, 7, 64, 72, 3, 3, (1, 1), (1, 1), (1, 1)),     # images end inside a tile
        (1, 20, 18, 128, 64, 3, 3, (1, 1), (1, 1), (1, 1)),  # several tiles
        (2, 11, 14, 72, 40, 3, 5, (2, 1), (1, 2), (1, 1)),   # C neither a k-tile nor an odd chunk count
        (1, 15, 13, 24, 136, 5, 3, (1, 2), (2, 0), (1, 1)),  # several column tiles
        (3, 7, 7, 16, 8, 1, 1, (2, 2), (0, 0), (1, 1)),      # strides that leave rows out, K below a k-tile
        (1, 17, 12, 40, 24, 3, 2, (1, 1), (2, 1), (2, 3)),   # dilation
        (5, 4, 3, 8, 16, 2, 2, (1, 1), (1, 1), (1, 1))]      # one chunk per tap, many images in a tile
EMU = [((256, 64, 3), "f16", 0), ((128, 128, 2), "f16", 0), ((128, 64, 3), "f16", 0), ((64, 128, 2), "bf16", 0),
       ((64, 64, 2), "f16", 0), ((256, 64, 2), "bf16", 1), ((128, 128, 3), "f16", 1), ((128, 64, 2), "bf16", 1),
       ((64, 64, 2), "f16", 1)]


def _case(g, dt, krsc):
    N, H, W, C, K, R, S, stride, pad, dil = g
    x = wl.small_ints((N, H, W, C), dt, 9700 + C)
    w = wl.small_ints((R, S, C, K), dt, 9800 + K)
    ref = oracle.conv2d(wl.bits(x), wl.bits(w), ODT[dt], stride, pad, dil)
    bias = torch.arange(K, dtype=torch.float32) % 5 - 2
    ref = oracle.epilogue(ref.reshape(-1, K), 0.5, bias.double().numpy(), 1).reshape(ref.shape)
    return x, w.permute(3, 0, 1, 2).contiguous() if krsc else w, bias, ref


def _run(x, w, y, g, bias, krsc, s, **kw):
    al.alcop_conv2d_igemm_dilated(x, w, y, g[7], g[8], g[9], 0.5, bias, 1, bool(krsc), s, **kw)


@pytest.mark.parametrize("tile,dt,krsc", EMU)
def test_exact_and_in_bounds_on_the_cpu_model(tile, dt, krsc):
    for n, g in enumerate(GEOM):
        x, w, bias, ref = _case(g, dt, krsc)
        y = torch.full(ref.shape, float("nan"))
        errs = emu.call(_run, x, w, y, g, bias, krsc, _sched(tile), reads=[x, w, bias],
                        writes=[y], policy=emu.POLICIES[n % 4])
        assert not errs, (g, errs[:4])
        assert np.array_equal(y.double().numpy(), ref), g


@pytest.mark.parametrize("mutation", [1, 2, 3])
def test_planted_synchronisation_mistakes_are_noticed(mutation):
    x, w, bias, ref = _case(GEOM[1], "f16", 0)
    y = torch.full(ref.shape, float("nan"))
    errs = emu.call(_run, x, w, y, GEOM[1], bias, 0, _sched((128, 64, 3)), reads=[x, w, bias],
                    writes=[y], policy=(1, 0), mutation=mutation)
    assert errs or not np.array_equal(y.double().numpy(), ref)


def test_non_finite_data_and_refusals():
    # chunks past K meet zero weights: they must be zeros, not neighbouring pixels (0 * inf)
    g = GEOM[0]
    x, w, bias, ref = _case(g, "f16", 0)
    x[1, 4, 3, 5] = float("inf")
    want = torch.nn.functional.conv2d(x.float().permute(0, 3, 1, 2), w.float().permute(3, 2, 0, 1), padding=1)
    want = torch.isfinite(want).permute(0, 2, 3, 1)
    y = torch.full(ref.shape, float("nan"))
    emu.call(al.alcop_conv2d_igemm, x, w, y, g[7], g[8], _sched((128, 64, 3)), reads=[x, w], writes=[y])
    assert torch.equal(torch.isfinite(y), want)
    big = wl.small_ints((1, 4, 1500, 64), "f16", 105)              # the halo of a 3 x 3 filter: too much LDS
    yb = torch.zeros(1, 4, 1500, 72, dtype=torch.float16)
    with pytest.raises(al.AlcopError) as e:
        emu.call(al.alcop_conv2d_igemm, big, w, yb, (1, 1), (1, 1), _sched((64, 64, 2)), reads=[big, w], writes=[yb])
    assert e.value.code == al.ERR_SCHED
    with emu._swapped():
        gemm = al.problem(al.OP_GEMM, 128, 64, 64, al.F16, al.F16)
        assert al.alcop_sched_supported(gemm, _sched((64, 64, 2))) == al.ERR_SCHED


# one problem description (M = 128, K = 576, 64 channels), four geometries: what a patch kernel may
# serve differs, so the library's pick must follow the call and not the problem
SAME = [(2, 8, 8, 64, 72, 3, 3, (1, 1), (1, 1), (1, 1)), (2, 16, 16, 64, 72, 3, 3, (2, 2), (1, 1), (1, 1)),
        (1, 2, 64, 64, 72, 3, 3, (1, 1), (1, 1), (1, 1)), (2, 8, 8, 64, 72, 3, 3, (1, 1), (2, 2), (2, 2))]


@pytest.mark.parametrize("krsc", [0, 1])
def test_default_pick_on_the_cpu_model(krsc):
    for n, g in enumerate(SAME + GEOM + SAME[::-1]):
        x, w, bias, ref = _case(g, "f16", krsc)
        y = torch.full(ref.shape, float("nan"))
        errs = emu.call(_run, x, w, y, g, bias, krsc, None, reads=[x, w, bias], writes=[y], policy=emu.POLICIES[n % 4])
        assert not errs, (g, errs[:4])
        assert np.array_equal(y.double().numpy(), ref), g


def test_a_loaded_schedule_wins_over_the_pick(tmp_path):
    # ... and one that this geometry cannot use gives way to the pick
    g = SAME[1]
    f = tmp_path / "cache"
    f.write_text("2 1 128 72 576 0 0 0 2 64 : 128 64 64 64 32 2 2 0 1 0 1\n")
    x, w, bias, ref = _case(g, "f16", 0)
    with emu._swapped():
        assert al.alcop_cache_load(str(f)) == 1
        prob = al.problem(al.OP_CONV2D, 128, 72, 576, al.F16, al.F32, conv_C=64)
        assert al.alcop_sched_auto(prob).variant == 1
    for g in SAME[:2]:                             # stride 1 takes it, stride 2 cannot
        x, w, bias, ref = _case(g, "f16", 0)
        y = torch.full(ref.shape, float("nan"))
        errs = emu.call(_run, x, w, y, g, bias, 0, None, reads=[x, w, bias], writes=[y])
        assert not errs and np.array_equal(y.double().numpy(), ref)


@pytest.mark.parametrize("tile", [(256, 64, 3), (128, 128, 2), (128, 64, 3), (64, 64, 2)])
def test_windows_that_overlap(tile, tmp_path, monkeypatch, capfd):
    # an RGB image laid out as two pixels per chunk: the gather's pixels are 8 elements apart, its windows
    # 32 elements long (224 deep with 7 filter rows); the schedule is loaded for that inner product
    N, H, W, C, K, R, S, stride, pad = 2, 13, 14, 3, 64, 7, 7, (2, 2), (3, 3)
    x, w = wl.small_ints((N, H, W, C), "f16", 9103), wl.small_ints((R, S, C, K), "f16", 9264)
    ref = oracle.conv2d(wl.bits(x), wl.bits(w), oracle.F16, stride, pad)
    f = tmp_path / "cache"
    f.write_text("2 1 98 64 224 0 0 0 0 32 : %s\n" % " ".join(map(str, _sched(tile).key())))
    y = torch.full(ref.shape, float("nan"), dtype=torch.float16)
    ws = torch.empty(al.alcop_conv2d_unaligned_workspace_bytes(N, H, W, C, K, R, S, stride, pad, (1, 1), al.F16),
                     dtype=torch.uint8)
    monkeypatch.setenv("ALCOP_LOG", "1")
    with emu._swapped():
        assert al.alcop_cache_load(str(f)) == 1
    errs = emu.call(al.alcop_conv2d_igemm_unaligned, x, w, y, ws, stride, pad, reads=[x, w], writes=[y, ws])
    assert "variant 4" in capfd.readouterr().err
    assert not errs, errs[:4]
    assert np.array_equal(y.double().numpy(), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("dt,krsc", [("f16", 0), ("f16", 1), ("bf16", 0)])
def test_default_pick_on_the_gpu(dt, krsc):
    # few tiles, many, patches, odd channels: every kind of kernel the pick knows
    for g in SAME + GEOM + [(8, 28, 28, 64, 64, 3, 3, (1, 1), (1, 1), (1, 1)), (3, 14, 14, 256, 192, 3, 3, (1, 1), (1, 1), (1, 1)),
                            (2, 33, 31, 288, 64, 5, 5, (1, 1), (2, 2), (1, 1)), (16, 40, 40, 32, 136, 1, 1, (1, 1), (0, 0), (1, 1))]:
        x, w, bias, ref = _case(g, dt, krsc)
        y = torch.full(ref.shape, float("nan"), device="cuda")
        _run(x.cuda(), w.cuda(), y, g, bias.cuda(), krsc, None)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().double().numpy(), ref), g


@pytest.mark.gpu
@pytest.mark.parametrize("krsc", [0, 1])
@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("tile", [(256, 64, 2), (256, 64, 3), (128, 128, 2), (128, 128, 3), (128, 64, 2), (128, 64, 3),
                                  (64, 128, 2), (64, 64, 2)])
def test_exact_on_the_gpu(tile, dt, krsc):
    for g in GEOM + [(3, 14, 14, 256, 192, 3, 3, (1, 1), (1, 1), (1, 1))]:
        x, w, bias, ref = _case(g, dt, krsc)
        for out in (torch.float32, TDT[dt]):
            y = torch.full(ref.shape, float("nan"), dtype=out, device="cuda")
            try:
                _run(x.cuda(), w.cuda(), y, g, bias.cuda(), krsc, _sched(tile))
            except al.AlcopError as e:            # the patch of 256 channels does not fit beside this ring
                assert e.code == al.ERR_SCHED and g[3] == 256, g
                continue
            torch.cuda.synchronize()
            want = torch.from_numpy(ref).to(out).double().numpy()
            assert np.array_equal(y.cpu().double().numpy(), want), (g, out)
