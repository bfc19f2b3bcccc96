"""Every path from a matrix instruction to the first use of its result, in the
built library, is as long as the hardware asks for.

The result of a matrix instruction is not interlocked against vector and
memory instructions: the compiler has to put enough instructions (or s_nop)
in between.  It was once found one short on the taken side of a branch behind
the last of a chain, and the kernel read old values.  So the distances are
counted here over all paths, taken branches included."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1705_09776_amd as cd

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if p and os.path.exists(p)), None)

# Wait states from issue to the first vector or memory use of the result: the
# instruction's passes and 4 (16-bit operands), or 2 (32-bit).
NEED = {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_16x16x16_bf16": 8, "v_mfma_f32_4x4x1_16b_f32": 4,
        "v_mfma_f32_16x16x4_f32": 10, "v_mfma_f32_32x32x2_f32": 18}


def _registers(operand):
    m = re.fullmatch(r"-?\|?([va])(?:\[(\d+):(\d+)\]|(\d+))\|?", operand)
    if not m:
        return set()
    lo, hi = (int(m[2]), int(m[3])) if m[2] else (int(m[4]), int(m[4]))
    return {(m[1], i) for i in range(lo, hi + 1)}


def _functions(path):
    """name -> [(address, opcode, operands)] of a code object."""
    text = subprocess.run([OBJDUMP, "-d", path], capture_output=True, text=True, check=True).stdout
    out, cur = {}, None
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if m:
            cur = out.setdefault(m[1], [])
            continue
        m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):", line)
        if m and cur is not None:
            cur.append((int(m[3], 16), m[1], [x.strip().split(" ")[0] for x in m[2].split(",")] if m[2] else []))
    return out


def _shortest(code, start, result):
    """Wait states from code[start] to the first non-matrix instruction that touches its result, over all paths."""
    at = {addr: i for i, (addr, _, _) in enumerate(code)}
    best, seen, todo = 99, {}, [(start + 1, 0)]
    while todo:
        i, waits = todo.pop()
        if i >= len(code) or waits >= best or waits > 24 or seen.get(i, 99) <= waits:
            continue
        seen[i] = waits
        addr, op, args = code[i]
        if any(_registers(a) & result for a in args):
            if not op.startswith("v_mfma"):   # (a chain of matrix instructions has rules of its own)
                best = waits
            continue
        step = int(args[0], 0) + 1 if op == "s_nop" else 1
        if op in ("s_endpgm", "s_setpc_b64"):
            continue
        if op.startswith(("s_cbranch", "s_branch")):
            offset = int(args[0], 0)
            offset -= 0x10000 if offset >= 0x8000 else 0
            todo.append((at[addr + 4 + 4 * offset], waits + 1))
            if op == "s_branch":
                continue
        todo.append((i + 1, waits + step))
    return best


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_results_are_not_used_too_early(tmp_path):
    if not os.path.exists(cd.LIB_PATH):
        cd.build()
    lib = shutil.copy(cd.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], capture_output=True, check=True, cwd=tmp_path)
    objects = [str(tmp_path / f) for f in os.listdir(tmp_path) if f.endswith("gfx950")]
    found, early = {}, []
    for path in objects:
        for name, code in _functions(path).items():
            for i, (_, op, args) in enumerate(code):
                if op.startswith("v_mfma"):
                    assert op in NEED, op
                    waits = _shortest(code, i, _registers(args[0]))
                    found[op] = min(found.get(op, 99), waits)
                    if waits < NEED[op]:
                        early.append((name, op, hex(code[i][0]), waits))
    assert set(found) == set(NEED)   # the library's kernels were looked at
    assert not early, early
