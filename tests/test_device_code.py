"""The library's own device code, disassembled: a buffer load that writes LDS stands in inline assembly, where the compiler's pass that keeps the required wait
states apart does not look.  A vector-memory instruction may read a scalar register no sooner than five wait states after a vector
instruction (v_readfirstlane, v_readlane, a compare, an addition's carry) wrote it: gfx950 does not hold the read back by itself."""
import os
import re
import struct
import subprocess

import pytest

from paper_1709_05011_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    blob = open(path, "rb").read()
    at = blob.find(BUNDLE)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + 24)
        pos = at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, pos)
            if size and b"gfx950" in blob[pos + 24:pos + 24 + length]:
                yield blob[at + offset:at + offset + size]
            pos += 24 + length
        at = blob.find(BUNDLE, at + 1)


def scalars(operand):
    m = re.fullmatch(r"s(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
    if not m:
        return set()
    return {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))


def early_reads(lines):
    """(LDS loads, those that read a scalar register too soon) of a listing, instruction by instruction in address order."""
    loads, bad, before, kernel = 0, [], [], None
    for line in lines:
        if line.startswith("<"):
            kernel, before = line, []
            continue
        op, _, rest = line.split("//")[0].strip().partition(" ")
        ops = rest.split(",")
        if op.startswith("buffer_load") and re.search(r"\blds\b", rest):
            loads += 1
            used, waits = scalars(ops[1]) | scalars(ops[2].split()[0]), 0
            for o, r in reversed(before):
                if waits >= 5 or not used:
                    break
                wrote = set()
                if o.startswith(("v_readfirstlane", "v_readlane", "v_cmp")):
                    wrote = scalars(r[0])
                elif o.startswith("v_") and "_co_" in o:
                    wrote = scalars(r[1])
                if wrote & used:
                    bad.append((kernel, line.strip(), waits))
                    break
                if o.startswith("s_") and not o.startswith(("s_cmp", "s_nop", "s_waitcnt", "s_barrier", "s_branch", "s_cbranch")):
                    used -= scalars(r[0])                          # written again by the scalar unit
                waits += int(r[0], 0) + 1 if o == "s_nop" else 1
        before = before[-8:] + [(op, ops)]
    return loads, bad


def test_listing_reader():
    load = ["s_mov_b32 m0, s5", "s_nop 0", "buffer_load_dwordx4 v5, s[12:15], s4 offen lds"]
    assert early_reads(["v_readfirstlane_b32 s4, v6"] + load)[1]
    assert early_reads(["v_readlane_b32 s15, v6, 1", "s_nop 1"] + load)[1]
    assert not early_reads(["v_readfirstlane_b32 s4, v6", "s_nop 2"] + load)[1]
    assert not early_reads(["v_readfirstlane_b32 s4, v6", "s_lshl_b32 s4, s4, 7"] + load)[1]
    assert not early_reads(["v_readfirstlane_b32 s6, v6"] + load)[1]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_scalar_operands_of_lds_loads_have_their_wait_states(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    loads, bad = 0, []
    for i, code in enumerate(code_objects(build.LIB)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(code)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)], capture_output=True, text=True, check=True).stdout
        n, b = early_reads(text.splitlines())
        loads, bad = loads + n, bad + b
    assert loads > 1000, loads
    assert not bad, bad[:5]
