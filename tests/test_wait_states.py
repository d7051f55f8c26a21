"""The machine code of the kernels: the waits that the hardware leaves to software, and registers.

A vector-memory instruction may read a scalar register only five wait states after the vector
instruction that wrote it.  The compiler keeps that distance for its own instructions but does not
look into inline asm, where the direct-to-LDS loads are: with a shorter one a load can take a stale
base address, which is a fault now and then and nothing that results show.

A vector instruction may write the data registers of a store wider than 8 bytes only two wait states
after it.  The stores that are written in inline asm bring both along: what follows them is the
compiler's choice.

The result of a matrix instruction may be read, or overwritten, only so many wait states after it: four more
than it has passes.  The compiler keeps that distance within a block of code, but where several ways lead to
the reading instruction it can miss the shortest: a partial sum without its last terms, always in the same lanes."""
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


STORE_WAIT = 2


def _vectors(operand):
    m = re.match(r"v\[(\d+):(\d+)\]|v(\d+)\b", operand.strip())
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def store_violations(asm):
    """(stores of more than 8 bytes from inline asm, those stores of any origin whose data registers are
    written too early, or, from inline asm, that do not bring the wait along).  Only the asm writes
    through (sc1)."""
    code = [t.strip() for t in asm.splitlines()]
    code = [t for t in code if t and t[0] not in ".;" and t[-1] != ":"]
    parts = lambda t: (t.partition(" ")[0], t.partition(" ")[2].split(","), t)
    seen, bad = 0, []
    for i, t in enumerate(code):
        if not re.match(r"(global|flat|scratch|buffer)_store_dwordx[34] ", t):
            continue
        op, args, t = parts(t)
        if re.search(r"\bsc1\b", t):
            seen += 1
            o, a, _ = parts(code[i + 1])
            if o != "s_nop" or int(a[0], 0) + 1 < STORE_WAIT:
                bad.append("no wait of its own: " + t)
        data = _vectors(args[0] if op.startswith("buffer_") else args[1])
        waited = 0
        for o, a, text in map(parts, code[i + 1:i + 1 + STORE_WAIT]):
            if waited >= STORE_WAIT or o.startswith(("s_cbranch", "s_branch", "s_endpgm")):
                break
            if o.startswith("v_") and _vectors(a[0]) & data:
                bad.append("%d wait states: %s ... %s" % (waited, t, text))
                break
            waited += int(a[0], 0) + 1 if o == "s_nop" else 1
    return seen, bad


def test_the_scan_finds_early_writes_of_stored_registers():
    store, through = "\tglobal_store_dwordx4 v8, v[4:7], s[0:1]", "\tglobal_store_dwordx4 v[8:9], v[4:7], off sc1"
    write, other = "\tv_mov_b32_e32 v6, 0", "\tv_mov_b32_e32 v8, 0"
    for code, n in (([store, write], 1), ([store, "\ts_nop 0", write], 1), ([store, "\ts_nop 1", write], 0),
                    ([store, other, other, write], 0), ([through, "\ts_nop 1", write], 0),
                    ([through, "\ts_nop 0", "\ts_or_b64 exec, exec, s[2:3]", write], 1),
                    (["\tglobal_store_dwordx2 v8, v[6:7], s[0:1]", write], 0),
                    (["\tbuffer_store_dwordx4 v[4:7], v0, s[0:3], 0 offen", write], 1)):
        assert len(store_violations("\n".join(code))[1]) == n, code


MATRIX_WAIT = {"32x32x16": 8 + 4, "16x16x32": 4 + 4}
REGISTER = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))(?![\w\[])")
CODE = re.compile(r"\t(\S+)(?: (.*?))? *// ([0-9A-F]+):(?:.*<[^>]*\+0x([0-9a-f]+)>)?")


def _used(operands):
    return {(m[1], r) for m in REGISTER.finditer(operands)
            for r in ([int(m[4])] if m[4] else range(int(m[2]), int(m[3]) + 1))}


def matrix_violations(asm, base):
    """(matrix instructions of a function at `base`, uses of their results that come too early on some way)."""
    code, at = [], {}
    for m in map(CODE.match, asm.splitlines()):
        if m:
            at[int(m[3], 16)] = len(code)
            code.append((m[1], m[2] or "", base + int(m[4], 16) if m[4] else None))
    seen, bad, used = 0, [], {}
    for i, (op, args, _) in enumerate(code):
        if not op.startswith("v_mfma"):
            continue
        seen += 1
        limit = next(n for shape, n in MATRIX_WAIT.items() if shape in op)
        result = _used(args.split(", ")[0])
        ways, least = [(i + 1, 0)], {}
        while ways:
            j, waited = ways.pop()
            if waited >= limit or least.get(j, limit) <= waited:
                continue
            least[j] = waited
            o, a, target = code[j]
            if j not in used:
                used[j] = _used(a)
            if o.startswith("v_mfma"):
                d, x, y, _ = a.split(", ", 3)
                early = (_used(x) | _used(y)) & result
                over = early or _used(d) & result            # accumulates, or takes the registers over
            else:
                early = over = used[j] & result
            if early:
                bad.append("%d of %d wait states: %s %s ... %s %s" % (waited, limit, op, args, o, a))
            if over or o == "s_endpgm":
                continue
            waited += int(a, 0) + 1 if o == "s_nop" else 1
            if target is not None and o.startswith(("s_branch", "s_cbranch")):
                ways.append((at[target], waited))
            if o != "s_branch":
                ways.append((j + 1, waited))
    return seen, bad


def test_the_scan_follows_a_result_over_branches():
    matrix = "v_mfma_f32_32x32x16_f16 a[0:15], v[20:23], v[24:27], a[0:15]"
    branch, read = "s_cbranch_scc1 3 <f+0x%x>", "v_accvgpr_read_b32 v1, a15"
    wait, other = "s_nop 10", "v_accvgpr_read_b32 v1, a16"
    for code, n in (([matrix, read], 1), ([matrix, "s_nop 11", read], 0), ([matrix, "s_nop 10", read], 1),
                    ([matrix, branch % 0x10, wait, wait, read], 1),                   # straight there
                    ([matrix, branch % 0x8, wait, other, read], 0), ([matrix, matrix, wait, "s_nop 0", read], 0),
                    ([matrix, "v_mfma_f32_16x16x32_bf16 v[0:3], a[12:15], v[4:7], 0"], 1),
                    ([matrix, "ds_write_b128 v9, a[0:3]"], 1), ([matrix, "s_endpgm", read], 0)):
        text = "\n".join("\t%s // %012X: 00000000 %s" % (t.split(" <")[0], 0x100 + 4 * k, "<" + t.split(" <")[1] if " <" in t else "")
                         for k, t in enumerate(code + ["s_endpgm"]))
        seen, bad = matrix_violations(text, 0x100)
        assert seen == sum("mfma" in t for t in code) and len(bad) == n, (code, bad)


def late_restores(asm):
    """Vector registers restored between the end of a branch on lanes and the restoring of the lane mask.

    Such a write reaches only the lanes of the inner mask.  Where the compiler has to reload a register
    that the branch used for something else, the other lanes keep what the branch left there."""
    lines, targets = [], set()
    for line in asm.splitlines():
        m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):", line)
        if m:
            lines.append((int(m[3], 16), m[1], m[2]))
            if m[1] == "s_cbranch_execz":
                n = int(m[2])
                targets.add(lines[-1][0] + 4 + 4 * (n - 65536 if n >= 32768 else n))
    bad, written, ended = [], [], False
    for address, op, args in lines:
        if address in targets or op.startswith("global_store"):
            ended, written = True, written if address in targets else []
        if op == "s_or_b64" and args.startswith("exec, exec"):
            bad += ["%s ahead of %s %s" % (written[0], op, args)] if ended and written else []
            ended, written = False, []
        elif "exec" in args or op.startswith(("s_cbranch", "s_branch", "s_endpgm")):
            ended, written = False, []
        elif ended and re.match(r"scratch_load|v_mov_b|v_accvgpr_", op) and re.search(r",.*\b([va][\d\[]|off)", args):
            written.append("%s %s" % (op, args))       # a copy or a reload, not a new value
    return bad


def test_the_scan_finds_late_restores():
    code = """
\ts_and_saveexec_b64 s[16:17], vcc                       // 000000000100:
\ts_cbranch_execz 7                                      // 000000000104: <k+0x24>
\tv_lshl_add_u64 v[254:255], v[18:19], 2, s[14:15]       // 000000000108:
\ts_and_b64 exec, exec, vcc                              // 000000000110:
\ts_cbranch_execz 2                                      // 000000000114: <k+0x20>
\tglobal_store_dwordx4 v[254:255], v[14:17], off nt      // 000000000118:
\t%s                                                     // 000000000120:
\ts_or_b64 exec, exec, s[16:17]                          // 000000000124:
"""
    assert len(late_restores(code % "v_mov_b32_e32 v255, v26")) == 1
    assert not late_restores(code % "s_mov_b32 s4, 0")


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
    tiles = re.findall(r"^[0-9a-f]+ <\w*Cfg\w*>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", asm, re.M | re.S)
    code = re.sub(r"//.*|<.*>:", "", asm)
    seen, early = 0, []
    for m in re.finditer(r"^([0-9a-f]+) <(\w+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", asm, re.M | re.S):
        n, bad = matrix_violations(m[3], int(m[1], 16))
        seen += n
        early += [m[2] + ": " + t for t in bad]
    return violations(code), [b for t in tiles for b in late_restores(t)], len(tiles), (seen, early), store_violations(code)


@pytest.fixture(scope="module")
def scans(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    files = []
    for i, code in enumerate(_code_objects(b.LIB)):
        files.append(str(tmp_path_factory.mktemp("code") / ("%d.co" % i)))
        open(files[-1], "wb").write(code)
    assert len(files) >= 20
    with cf.ProcessPoolExecutor(max_workers=8, mp_context=multiprocessing.get_context("spawn")) as ex:
        return list(ex.map(_scan, files))


def test_loads_keep_their_distance_from_the_descriptor(scans):
    assert sum(n for (n, _), *_ in scans) > 100000
    bad = [v for (_, vs), *_ in scans for v in vs]
    assert not bad, (len(bad), bad[:3])


def test_no_register_is_restored_under_an_inner_lane_mask(scans):
    assert sum(n for _, _, n, *_ in scans) > 1000
    bad = [v for _, vs, *_ in scans for v in vs]
    assert not bad, (len(bad), bad[:3])


def test_stored_registers_keep_their_values_until_they_are_read(scans):
    assert sum(n for *_, (n, _) in scans) > 1000
    bad = [v for *_, (_, vs) in scans for v in vs]
    assert not bad, (len(bad), bad[:3])


def test_matrix_results_are_complete_when_they_are_used(scans):
    assert sum(n for *_, (n, _), _ in scans) > 10000
    bad = [v for *_, (_, vs), _ in scans for v in vs]
    assert not bad, (len(bad), bad[:3])


READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _registers(path):
    """{tile-at-a-time kernel's template arguments: (vector registers, bytes of scratch)}"""
    notes = subprocess.run([READELF, "--notes", path], check=True, stdout=subprocess.PIPE, text=True).stdout
    out = {}
    for block in notes.split("- .agpr_count:")[1:]:
        value = lambda key: re.search(key + r":\s+(\S+)", block)[1]
        cfg = re.search(r"4KCfgI([Li\dE]+)EE", value(r"\.name"))
        if cfg:
            out[tuple(map(int, re.findall(r"Li(\d+)E", cfg[1] + "E")))] = (
                int(value(r"\.vgpr_count")), int(value(r"\.private_segment_fixed_size")))
    return out


def test_the_bias_of_a_tile_takes_no_registers_that_the_kernel_lacks(tmp_path):
    # held whole it took two blocks of 64 x 96 waves per compute unit to one (more than 256
    # registers), and 128 x 128 waves to 400 - 964 bytes of scratch (280 - 392 without)
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    kernels = {}
    for code in _code_objects(b.LIB):
        path = str(tmp_path / "code.co")
        open(path, "wb").write(code)
        kernels.update(_registers(path))
    seen = set()
    for (_, _, _, _, wm, wn, _, r, _, _, _, a_km, *_), (vgprs, scratch) in kernels.items():
        if a_km:
            continue               # A stored K x M keeps the array
        seen.add((wm, wn))
        if (wm, wn) == (64, 96):
            assert vgprs <= 256
        assert scratch <= (0 if (wm, wn) != (128, 128) else 392 if r > 2 else 296), (wm, wn, r)
    assert {(64, 96), (128, 96), (128, 128), (64, 64)} <= seen
