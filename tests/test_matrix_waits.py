"""Wait states between the matrix instructions of the built library and the first
vector or memory instruction that touches their results.

The hardware does not hold such an instruction back: the compiler counts wait
states (one per instruction, n + 1 for s_nop n) along every way from the matrix
instruction and fills what is missing.  Where a reader can be reached both
directly and over a short branch it has been seen to count the longer way only.
This test counts every way in the disassembly of libspire.so, and checks its own
counting on listings with a known answer."""
import collections
import os
import re
import shutil
import subprocess

import pytest

from paper_2504_06419_amd import spire

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
# wait states before a result may be read or overwritten: 4 passes + 4, 8 passes + 2
NEED = {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_16x16x32_f16": 8, "v_mfma_f32_16x16x4_f32": 10}


def _registers(operand):
    m = re.match(r"^[-|]*([va])(\d+)\b", operand)
    if m:
        return {(m.group(1), int(m.group(2)))}
    m = re.match(r"^[-|]*([va])\[(\d+):(\d+)\]", operand)
    return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)} if m else set()


def parse(listing):
    """{function: [(mnemonic, operand registers, operands, address, branch target)]}"""
    functions, cur, start = {}, None, 0
    for line in listing.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
        if m:
            cur, start = functions.setdefault(m.group(2), []), int(m.group(1), 16)
            continue
        m = re.match(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):(?: [0-9A-F]+)*(?: <\S+?(?:\+0x([0-9a-f]+))?>)?\s*$", line)
        if m and cur is not None:
            ops = [o.strip() for o in re.split(r",(?![^\[]*\])", m.group(2)) if o.strip()]
            target = start + int(m.group(4) or "0", 16) if "branch" in m.group(1) else None
            cur.append((m.group(1), [_registers(o) for o in ops], ops, int(m.group(3), 16), target))
    return functions


def shortfalls(code):
    """[(matrix instruction, reader, wait states between them, needed)] of one function."""
    at = {ins[3]: i for i, ins in enumerate(code)}
    found = []
    for i, (name, regs, _, addr, _) in enumerate(code):
        if not name.startswith("v_mfma"):
            continue
        need, result = NEED[name], regs[0]
        todo, best = collections.deque([(i + 1, 0)]), {}
        while todo:
            j, waits = todo.popleft()
            if j >= len(code) or waits >= need or best.get(j, need) <= waits:
                continue
            best[j] = waits
            op, opregs, ops, opaddr, target = code[j]
            if op.startswith("v_mfma"):
                if (opregs[1] | opregs[2]) & result:
                    found.append((hex(addr), f"{op} {hex(opaddr)}", waits, need))
                if any(r & result for r in opregs):
                    continue                       # accumulates in order, or overwrites
            elif op.startswith(("v_", "global_", "ds_", "buffer_", "flat_", "scratch_")):
                if any(r & result for r in opregs):
                    found.append((hex(addr), f"{op} {hex(opaddr)}", waits, need))
                    continue
            if op == "s_endpgm":
                continue
            waits += int(ops[0], 0) + 1 if op == "s_nop" else 1
            if target is not None:
                todo.append((at[target], waits))
            if op != "s_branch":
                todo.append((j + 1, waits))
    return found


def _listing(body):
    return "0000000000000000 <f>:\n" + "".join(f"\t{ins:60s} // {4 * i:012X}: 00000000{tgt}\n"
                                               for i, (ins, tgt) in enumerate(body))


MFMA = ("v_mfma_f32_16x16x4_f32 v[0:3], v8, v9, v[0:3]", "")
READ = ("v_add_f32_e32 v10, v2, v11", "")
OTHER = ("v_mov_b32_e32 v12, v13", "")


@pytest.mark.parametrize("body,short", [
    ([MFMA, READ], 1), ([MFMA, ("s_nop 8", ""), READ], 1), ([MFMA, ("s_nop 9", ""), READ], 0),
    # a branch around ten other instructions: the direct way has two wait states
    ([MFMA, ("s_cbranch_scc1 11", " <f+0x30>")] + [OTHER] * 10 + [READ], 1),
    ([MFMA, ("s_nop 9", ""), ("s_cbranch_scc1 11", " <f+0x34>")] + [OTHER] * 10 + [READ], 0),
    ([MFMA, ("v_mfma_f32_16x16x4_f32 v[0:3], v8, v9, v[0:3]", ""), ("s_nop 9", ""), READ], 0),
    ([MFMA, ("v_mfma_f32_16x16x4_f32 v[4:7], v1, v9, v[4:7]", "")], 1),
    ([MFMA] + [OTHER] * 9 + [("global_store_dwordx4 v[20:21], v[0:3], off", "")], 1)])
def test_counting(body, short):
    code = parse(_listing(body))["f"]
    assert len(code) == len(body) and len(shortfalls(code)) == short


def test_library(tmp_path):
    objdump = os.path.join(LLVM, "llvm-objdump")
    if not os.path.exists(objdump) or not os.path.exists(spire.LIB_PATH):
        pytest.skip("needs llvm-objdump and the built library")
    lib = shutil.copy(spire.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([objdump, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    objects = sorted(p for p in os.listdir(tmp_path) if "gfx950" in p)
    assert objects
    kinds, bad = collections.Counter(), []
    for obj in objects:
        text = subprocess.run([objdump, "-d", "--mcpu=gfx950", str(tmp_path / obj)], check=True, capture_output=True,
                              text=True).stdout
        for name, code in parse(text).items():
            kinds.update(ins[0] for ins in code if ins[0].startswith("v_mfma"))
            bad += [(name,) + b for b in shortfalls(code)]
    print(dict(kinds))
    assert kinds["v_mfma_f32_16x16x4_f32"] > 100 and kinds["v_mfma_f32_16x16x32_bf16"] > 1000
    assert not bad, f"{len(bad)} short, first {bad[:3]}"
