"""The backward kernels on the CPU: every address inside its tensor, every barrier met by all, and
the one pass against the two passes and against sums in double, at the sizes where indexes can go wrong.

The kernels' own sources are compiled for the CPU with stand-ins for what the processor does across lanes
(tests/emulate); tensors lie between pages that may not be touched."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2208_08124_amd", "csrc")
HERE = os.path.join(ROOT, "tests", "emulate")
CLANG = shutil.which("clang++") or next((p for p in ("/opt/rocm/llvm/bin/clang++", "/opt/rocm/lib/llvm/bin/clang++")
                                         if os.path.exists(p)), None)

pytestmark = pytest.mark.skipif(CLANG is None, reason="no clang++ (vector types, 16-bit floats)")


def statement(m):
    """What stands in for an inline assembly statement."""
    s = m.group(0)
    if "load_lds" in s:
        size = 16 if "dwordx4" in s else 4
        to = "lds_byte_addr + more" if "(more)" in s else "lds_byte_addr"
        return f"emu::dma({'(const char*)sbase + voff' if 'sbase' in s else 'gptr'}, {to}, {size});"
    if "s_barrier" in s:
        return "emu::meet(emu::kWorkgroup);"
    return ";"  # waits, and values held in registers


def translate(text):
    text = re.sub(r"__attribute__\(\(address_space\(\d\)\)\)", "", text)
    text = re.sub(r'asm volatile\((?:[^;"]|"[^"]*")*\);', statement, text)
    text = text.replace("__shared__ uint32_t mailbox;", "uint32_t& mailbox = *(uint32_t*)(emu::lds + 159 * 1024);")
    text = re.sub(r"__shared__ __align__\(1024\) (\w+) (\w+)((?:\[\w+\])*);",
                  lambda m: f"auto& {m[2]} = *({m[1]}(*){m[3]})emu::lds;" if m[3] else f"{m[1]}& {m[2]} = *({m[1]}*)emu::lds;", text)
    assert "__shared__" not in text
    return text


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("emulate")
    os.mkdir(d / "translated")
    for f in ("bwd_fused_kernel.h", "bwd_kernels.h", "dropout.h", "item_feed.h", "kernel_args.h", "mfma_tiles.h"):
        (d / "translated" / f).write_text(translate(open(os.path.join(CSRC, f)).read()))
    subprocess.check_call([CLANG, "-O1", "-std=c++17", "-w", "-I", HERE, "-I", str(d), "-o", str(d / "backward"),
                           os.path.join(HERE, "backward.cpp")])
    return str(d / "backward")


def emulate(program, dtype, thr, heads, lengths, used=None, values="normal", slab_rows=2048, grid=8, edge=1):
    cmd = [program, dtype, str(thr), str(heads), str(grid), str(slab_rows), str(edge), values, ",".join(map(str, lengths))]
    if used is not None:
        cmd.append(",".join(map(str, used)))
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[:2000]
    out = {}
    for line in r.stdout.splitlines():
        w = line.split()
        out[w[0]] = float(w[1]) if len(w) == 2 else {"two": float(w[2]), "double": float(w[4]), "bad": (int(w[6]), int(w[7])),
                                                     "largest": float(w[9])}
    assert out["counters"] == 0
    return out


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("lengths,heads,used,thr,slab_rows", [
    ([1, 32, 33, 64, 65, 96, 128, 129, 256], 3, None, 0, 256),             # four, two and one head at a time, one left over
    ([3, 64, 17, 100, 31], 5, None, 64, 256),
    ([69] * 5, 2, [69, 1, 40, 33, 0], 0, 256),                             # one head at a time, of few queries: a partial
    ([20, 35, 100, 97], 2, [20, 3, 64, 97], 26, 256),                      #   block is the first that is requested
    ([257, 300, 512], 1, None, 0, 512),                                    # two sweeps
    ([385, 290], 1, [260, 33], 26, 512),
    ([290], 2, None, 0, 256),                                              # more rows than the buffer holds: parts of 256, the
    ([523], 1, None, 26, 256),                                             #   last of which is a partial block or two
])
def test_backward_stays_in_range_and_agrees(program, lengths, heads, used, thr, slab_rows, dtype):
    """The bounds: 4 times what rounding P and dS to the operand type leaves in these sums (4e-4 and 3e-3), for dQ and
    dK of the two kernels against each other, which round dP - D in another order, the same."""
    tol = 1.6e-3 if dtype == "f16" else 1.2e-2
    for edge in (1, 0):
        r = emulate(program, dtype, thr, heads, lengths, used, slab_rows=slab_rows, edge=edge)
        for g in ("dq", "dk", "dv"):
            assert r[g]["bad"] == (0, 0) and r[g]["two"] <= tol and r[g]["double"] <= tol, (g, r[g])
        assert r["dv"]["two"] == 0 and (thr == 0 or r["dk"]["two"] == 0)


@pytest.mark.parametrize("lengths,used", [([1] * 9, None), ([33, 40, 5, 70], None), ([69, 40], [33, 40]), ([300, 129], None)])
def test_key_places_without_a_key_add_nothing(program, lengths, used):
    """Every row attends to its sequence's last key alone, whose dP / (1 - p) = 524 288 is beyond f16's range, and half
    the scores are dropped: dS = P (dP - D) is 0, kept or not.  What stands behind the last key is a copy of it with a mask
    of its own, and its P (dP - D) would not be 0."""
    r = emulate(program, "f16", 128, 2, lengths, used, values="last")
    for g in ("dq", "dk", "dv"):
        assert r[g]["bad"] == (0, 0) and r[g]["two"] == 0, (g, r[g])
    assert r["dq"]["largest"] == 0 and r["dv"]["largest"] > 0
