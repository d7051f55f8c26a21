"""The waits that the hardware leaves to software, in the machine code of the kernels.

A vector-memory instruction may read a scalar register only five wait states after the vector
instruction that wrote it.  The compiler keeps that distance for its own instructions but does not
look into inline asm, where the direct-to-LDS loads are: with a shorter one a load can take a stale
base address, which is a fault now and then and nothing that results show."""
import concurrent.futures as cf
import multiprocessing
import os
import re
import struct
import subprocess

import pytest

from paper_2210_16691_amd import build as b

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT = 5


def _scalars(operand):
    m = re.match(r"s\[(\d+):(\d+)\]|s(\d+)\b", operand.strip())
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def violations(asm):
    """(vector-memory instructions seen, those that read a scalar register too early)."""
    seen, bad, past = 0, [], []
    for line in asm.splitlines():
        t = line.split(";")[0].strip()
        if not t or t[0] == "." or t.endswith(":"):
            continue
        op, _, rest = t.partition(" ")
        args = rest.split(",")
        if op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            seen += 1
            needs = set().union(*map(_scalars, args))
            waited = 0
            for o, a, text in reversed(past):
                if waited >= WAIT:
                    break
                written = a[:2] if "_co_" in o else a[:1]
                if o.startswith("v_") and set().union(*map(_scalars, written)) & needs:
                    bad.append("%d wait states: %s ... %s" % (waited, text, t))
                    break
                waited += int(a[0], 0) + 1 if o == "s_nop" else 1
        past = (past + [(op, args, t)])[-8:]
    return seen, bad


def test_the_scan_counts_wait_states():
    load = "\tbuffer_load_dwordx4 v5, s[16:19], 0 offen lds"
    move = "\ts_mov_b32 m0, s25"
    for between, n in (([move, "\ts_nop 0"], 1), ([move, "\ts_nop 2", "\tv_add_u32_e32 v1, s2, v1"], 0),
                       (["\tv_readfirstlane_b32 s20, v3"] + [move] * 3, 1), (["\ts_nop 4"], 0)):
        assert len(violations("\n".join(["\tv_readfirstlane_b32 s17, v4"] + between + [load]))[1]) == n


def _code_objects(path):
    """The gfx950 code objects bundled in a library."""
    data = open(path, "rb").read()
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        o = m.start()
        n, at = struct.unpack_from("<Q", data, o + 24)[0], o + 32
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            if b"gfx950" in data[at + 24:at + 24 + length]:
                yield data[o + offset:o + offset + size]
            at += 24 + length


def _scan(path):
    asm = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", "--no-show-raw-insn", path], check=True,
                         stdout=subprocess.PIPE, text=True).stdout
    return violations(re.sub(r"//.*|<.*>:", "", asm))


def test_loads_keep_their_distance_from_the_descriptor(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    files = []
    for i, code in enumerate(_code_objects(b.LIB)):
        files.append(str(tmp_path / ("%d.co" % i)))
        open(files[-1], "wb").write(code)
    assert len(files) >= 20
    with cf.ProcessPoolExecutor(max_workers=8, mp_context=multiprocessing.get_context("spawn")) as ex:
        found = list(ex.map(_scan, files))
    assert sum(n for n, _ in found) > 100000
    bad = [v for _, vs in found for v in vs]
    assert not bad, (len(bad), bad[:3])
