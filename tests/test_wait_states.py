"""The waits that the hardware leaves to software, in the machine code of the kernels.

A vector-memory instruction may read a scalar register only five wait states after the vector
instruction that wrote it.  The compiler keeps that distance for its own instructions but does not
look into inline asm, where the direct-to-LDS loads are: with a shorter one a load can take a stale
base address, which is a fault now and then and nothing that results show."""
import os
import re
import subprocess

import pytest

from paper_2210_16691_amd import build as b

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


@pytest.mark.parametrize("source", ["inst_f16_kn_mid.hip", "inst_nk_big.hip", "inst_convres_rsck.hip", "inst_ksplit.hip"])
def test_loads_keep_their_distance_from_the_descriptor(source, tmp_path):
    if not os.path.exists(b.HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path / "k.s"
    subprocess.run([b.HIPCC] + b.FLAGS + ["-x", "hip", "-S", "--cuda-device-only", os.path.join(b.CSRC, source), "-o", str(out)],
                   check=True, stderr=subprocess.DEVNULL)
    seen, bad = violations(out.read_text())
    assert seen > 100
    assert not bad, bad[:3]
