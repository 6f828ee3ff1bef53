"""Waits that gfx950 leaves to the program, looked for in the instructions of the built library.

The compiler places them between its own instructions, but not inside inline assembly, nor between an
instruction of its own and one that it does not see.  Two of them concern the transfers into LDS, which
are written as assembly: five wait states from a vector instruction that writes scalar registers to a
memory instruction that reads them, and one from a write of m0 to a transfer into LDS."""
import glob
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2208_08124_amd", "libfmha_varlen.so")
CSRC = os.path.join(ROOT, "paper_2208_08124_amd", "csrc")
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"

VMEM = re.compile(r"(global|buffer|scratch|flat)_")
VECTOR_TO_SCALAR = re.compile(r"v_(readlane|readfirstlane|cmp)")


def code_objects(path):
    """The gfx950 code objects of a library built by hipcc (one bundle per source file)."""
    data, magic = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length] and size:
                yield data[at + off:at + off + size]
            p += 24 + length
        at = data.find(magic, at + 24)


def registers(text):
    out = set()
    for a, b, c in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text):
        out |= set(range(int(a), int(b) + 1)) if a else {int(c)}
    return out


def short_waits(lines):
    """(kernel, instruction, what it waits too little for) of a disassembly."""
    found, transfers, kernel, before = [], 0, None, []
    for line in lines:
        m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if m:
            kernel, before = m.group(1), []
            continue
        text = line.split("//")[0].strip()
        if not text or text.endswith(":"):
            continue
        op, _, args = text.partition(" ")
        if VMEM.match(op):
            lds = "load_lds" in op or re.search(r"\blds\b", args)
            transfers += bool(lds)
            reads, states = registers(args), 0
            for o, a in reversed(before):
                if states >= 5:
                    break
                dst = a.split(",")[0]
                if lds and states < 1 and o.startswith("s_") and dst.strip() == "m0":
                    found.append((kernel, text, "m0"))
                if VECTOR_TO_SCALAR.match(o) and registers(dst) & reads:
                    found.append((kernel, text, f"{o} {a}"))
                elif o.startswith("s_") and not o.startswith("s_cmp"):
                    reads -= registers(dst)  # (written again by a scalar instruction, which is waited for)
                states += int(a, 0) + 1 if o == "s_nop" else 1
        before = before[-8:] + [(op, args.strip())]
    return found, transfers


def test_the_search_finds_what_it_is_for():
    head = ["0000000000001000 <k>:"]
    bad = ["v_readlane_b32 s5, v255, 18", "s_mov_b32 m0, s57", "global_load_lds_dwordx4 v194, s[4:5]"]
    assert [w for _, _, w in short_waits(head + bad)[0]] == ["m0", "v_readlane_b32 s5, v255, 18"]
    assert short_waits(head + bad[:2] + ["s_nop 2"] + bad[2:])[0] != []
    assert short_waits(head + bad[:2] + ["s_nop 3"] + bad[2:])[0] == []
    assert short_waits(head + bad[:1] + ["s_addc_u32 s5, s9, s5", "s_mov_b32 m0, s57", "s_nop 0"] + bad[2:])[0] == []


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built (run __graft_entry__.build())")
@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler for what was built here")
def test_transfers_wait_for_their_base_and_for_m0(tmp_path):
    transfers = 0
    for i, code in enumerate(code_objects(LIB)):
        f = tmp_path / f"{i}.co"
        f.write_bytes(code)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True, check=True).stdout
        found, n = short_waits(text.splitlines())
        assert not found, found[:10]
        transfers += n
    assert transfers > 500


def test_inline_assembly_holds_no_vector_arithmetic():
    """What a matrix instruction still reads or writes is known to the compiler alone."""
    for path in glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip")):
        for body in re.findall(r'asm volatile\("([^"]*)"', open(path).read()):
            assert not re.search(r"(^|[\s\\nt])v_\w+", body), (path, body)
