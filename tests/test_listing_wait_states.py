"""The listing of every kernel in the built bf16 library is walked for one hazard: a
vector instruction that reads a matrix-core result before it is written.  The hardware
does not wait there; the compiler inserts the wait states, but ROCm 7.2 left them out
behind a branch between the product and the first use (wrong g_z in some tiles).  From
every product, along the straight path and both sides of every branch, a read of its
result as a vector operand has to lie at least as many states on as the compiler puts
there on straight paths (gfx950: eight for the four passes of a bf16 product, 11 and,
for memory instructions, 18 for a float64 one).  (A product that only accumulates onto
the result waits by itself.)
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_11947_amd import build as B

OBJDUMP = os.path.join(os.path.dirname(os.path.dirname(B.hipcc())), "llvm", "bin", "llvm-objdump")
STATES = {"16x16x32_bf16": (8, 8), "16x16x4_f64": (11, 18)}  # before a vector, a memory instruction
LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]{12}):")
TARGET = re.compile(r"<(\w+?)(?:\+0x([0-9a-f]+))?>$")
REG = re.compile(r"\b([av])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def regs(text):
    out = set()
    for f, lo, hi, one in REG.findall(text):
        out.update((f, i) for i in ((int(one),) if one else range(int(lo), int(hi) + 1)))
    return out


def parse(text):
    """Instructions [(op, operands, branch target)] and their index by (address)."""
    code, at, start = [], {}, {}
    name = None
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]{16}) <(\w+)>:", line)
        if m:
            name = m.group(2)
            start[name] = int(m.group(1), 16)
            continue
        m = LINE.match(line)
        if not m:
            continue
        op, rest, addr = m.groups()
        target = None
        if op.startswith(("s_cbranch", "s_branch")):
            sym, off = TARGET.search(line).groups()
            target = (sym, int(off or "0", 16))
        at[int(addr, 16)] = len(code)
        code.append((op, rest, target, name))
    return [(op, rest, at.get(start[t[0]] + t[1]) if t else None, nm) for op, rest, t, nm in code]


def early_reads(code):
    found = []
    for i, (op, rest, _, name) in enumerate(code):
        if not op.startswith("v_mfma"):
            continue
        dst = regs(rest.split(",")[0])
        valu, memory = next(v for k, v in STATES.items() if k in op)
        stack, seen = [(i + 1, 0)], {}
        while stack:
            j, st = stack.pop()
            while j is not None and j < len(code) and st < memory:
                if seen.get(j, memory) <= st:
                    break
                seen[j] = st
                o, r, target, _ = code[j]
                if o == "s_endpgm":
                    break
                if o == "s_nop":
                    st += int(r, 0) + 1
                    j += 1
                    continue
                if o.startswith("s_cbranch"):
                    stack.append((target, st + 1))
                elif o == "s_branch":
                    j, st = target, st + 1
                    continue
                elif o.startswith("v_mfma"):
                    parts = r.split(", ")
                    if st < valu and dst & (regs(parts[1]) | regs(parts[2])):
                        found.append((name, i, op, j, o, st, valu))
                    if dst & regs(parts[0]):
                        break
                elif o.startswith(("v_", "ds_", "buffer_", "global_", "flat_", "scratch_")) and dst & regs(r):
                    need = valu if o.startswith("v_") else memory
                    if st < need:
                        found.append((name, i, op, j, o, st, need))
                    break
                st += 1
                j += 1
    return found


def test_walker_finds_an_early_read():
    """On a listing written here: a read two states on through a branch, none on the straight path."""
    text = "\n".join([
        "0000000000001000 <k>:",
        "\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], 0      // 000000001000: 0 0",
        "\ts_cbranch_scc1 3                                          // 000000001008: 0 <k+0x14>",
        "\ts_nop 6                                                   // 00000000100C: 0",
        "\tv_add_f32_e32 v12, v3, v13                                // 000000001010: 0",
        "\tv_add_f32_e32 v12, v2, v13                                // 000000001014: 0",
        "\ts_endpgm                                                  // 000000001018: 0",
    ])
    assert [(f[3], f[5]) for f in early_reads(parse(text))] == [(4, 1)]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump beside the compiler")
def test_no_kernel_reads_a_product_early(tmp_path):
    if not os.path.exists(B.lib_path()):
        B.build_all()
    lib = shutil.copy(B.lib_path(), tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    objects = [f for f in sorted(os.listdir(tmp_path)) if f.endswith("gfx950")]
    assert len(objects) == 3, objects
    products = 0
    for f in objects:
        text = subprocess.run([OBJDUMP, "-d", f], check=True, capture_output=True, text=True, cwd=tmp_path).stdout
        code = parse(text)
        products += sum(op.startswith("v_mfma") for op, _, _, _ in code)
        assert early_reads(code) == []
    assert products > 10000
