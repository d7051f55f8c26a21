"""What a saved and reloaded tuning cache does to calls without a schedule, on the CPU model."""
import re

import numpy as np
import torch

import emu_util as emu
import oracle
import paper_2210_16691_amd as al
import workloads as wl


def _tile(err):
    return re.findall(r"-> (tile .*) variant (\d)", err)[-1]


def test_the_librarys_own_picks_stay_picks_after_save_and_load(tmp_path, monkeypatch, capfd):
    # the entry of a convolution's problem description knows no image geometry: read back as if it had
    # been tuned it would keep the kernels with a resident patch from being picked
    N, H, W, C, K = 1, 13, 11, 16, 80
    x, w = wl.small_ints((N, H, W, C), "f16", 51), wl.small_ints((3, 3, C, K), "f16", 52)
    ref = oracle.conv2d(wl.bits(x), wl.bits(w), oracle.F16, (1, 1), (1, 1))
    f = str(tmp_path / "cache")
    monkeypatch.setenv("ALCOP_LOG", "1")

    def run():
        y = torch.full(ref.shape, float("nan"))
        assert not emu.call(al.alcop_conv2d_igemm, x, w, y, (1, 1), (1, 1), reads=[x, w], writes=[y])
        assert np.array_equal(y.double().numpy(), ref)
        return _tile(capfd.readouterr().err)

    first = run()
    assert first[1] == "4"
    prob = al.problem(al.OP_CONV2D, N * H * W, K, 9 * C, al.F16, al.F32, conv_C=C)
    with emu._swapped():
        plain = al.alcop_sched_auto(prob)
        assert plain.variant != 4
        n = al.alcop_cache_save(f)
        assert n >= 1 and al.alcop_cache_load(f) == n
        assert al.alcop_sched_auto(prob).key() == plain.key()
    assert run() == first
    # a tuned entry survives a file's pick of the same problem, and is one after its own save and load
    line = [t for t in open(f) if t.startswith("2 1 %d %d %d " % (N * H * W, K, 9 * C))]
    tuned = tmp_path / "tuned"
    other = [s for s in emu.space(prob) if s.key() != plain.key()][0]
    tuned.write_text("%s: %s\n" % (line[0].split(":")[0], " ".join(map(str, other.key()))))
    with emu._swapped():
        assert al.alcop_cache_load(str(tuned)) == 1 and al.alcop_cache_load(f) == n
        assert al.alcop_cache_save(f) == n and al.alcop_cache_load(f) == n
        assert al.alcop_sched_auto(prob).key() == other.key()
    assert run() != first


def _load(tmp_path, prob, sched):
    p = tmp_path / "entry"
    p.write_text("%d 1 %d %d %d %d %d %d %d %d : %s\n" % (prob.op, prob.M, prob.N, prob.K, prob.transA, prob.transB,
                                                         prob.in_, prob.out, prob.conv_C,
                                                         " ".join(map(str, sched.key()))))
    with emu._swapped():
        assert al.alcop_cache_load(str(p)) == 1


def test_unaligned_calls_find_the_entry_of_the_padded_problem(tmp_path, monkeypatch, capfd):
    monkeypatch.setenv("ALCOP_LOG", "1")
    # a convolution with few channels: the problem padded to 8, whatever layout the call would choose
    N, H, W, C, K = 1, 15, 19, 3, 40
    x, w = wl.small_ints((N, H, W, C), "f16", 53), wl.small_ints((7, 7, C, K), "f16", 54)
    ref = oracle.conv2d(wl.bits(x), wl.bits(w), oracle.F16, (2, 2), (3, 3))
    ws = torch.empty(al.alcop_conv2d_unaligned_workspace_bytes(N, H, W, C, K, 7, 7, (2, 2), (3, 3), (1, 1), al.F32),
                     dtype=torch.uint8)
    prob = al.problem(al.OP_CONV2D, ref.size // K, K, 49 * 8, al.F16, al.F32, conv_C=8)
    tiles = emu.space(prob)
    for entry in (None, tiles[0], tiles[-1]):
        if entry is not None:
            _load(tmp_path, prob, entry)
        y = torch.full(ref.shape, float("nan"))
        assert not emu.call(al.alcop_conv2d_igemm_unaligned, x, w, y, ws, (2, 2), (3, 3), reads=[x, w], writes=[y, ws])
        assert np.array_equal(y.double().numpy(), ref)
        err = capfd.readouterr().err
        if entry is None:
            assert "K 224 " in err
        else:
            assert "K 392 " in err and "tile %dx%dx%d waves" % entry.key()[:3] in err
    # a product with an odd number of rows: M rounded up to 8 (not stored K x M, the rows need no padding)
    M, N, K = 37, 29, 45
    A, B = wl.small_ints((M, K), "f16", 55), wl.small_ints((K, N), "f16", 56)
    prob = al.problem(al.OP_GEMM, 40, 32, 48, al.F16, al.F32)
    ws = torch.empty(al.alcop_unaligned_workspace_bytes(1, M, N, K, al.F32), dtype=torch.uint8)
    for entry in [s for s in emu.space(prob) if s.variant == 0][:2]:
        _load(tmp_path, prob, entry)
        y = torch.full((M, N), float("nan"))
        assert not emu.call(al.alcop_bmm_unaligned, A, B, y, ws, reads=[A, B], writes=[y, ws])
        assert np.array_equal(y.double().numpy(), oracle.gemm(wl.bits(A), wl.bits(B), oracle.F16))
        assert "tile %dx%dx%d waves %dx%d S%d R%d F%d" % entry.key()[:8] in capfd.readouterr().err
