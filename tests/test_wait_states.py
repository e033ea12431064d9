"""The wait states between a matrix product and a vector instruction that touches its result, in the built library, on every path: the
compiler counts them, but not always across a branch, and too few give wrong values now and then without an error."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2402_05099_amd import binding as hb

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
NEED = {"v_mfma_f32_16x16x32_bf16": 8, "v_mfma_f32_32x32x16_bf16": 12}      # instructions or s_nop counts between the two


def functions(listing):
    """{name: [(address, instruction, operands, branch target)]} of the functions with matrix products"""
    out, name, start = {}, None, 0
    for line in listing.splitlines():
        m = re.match(r"([0-9a-f]+) <(.+)>:$", line)
        if m:
            name, start = m.group(2), int(m.group(1), 16)
            out[name] = []
        elif name and "//" in line:
            text, note = line.split("//", 1)
            op, _, operands = text.strip().partition(" ")
            to = re.search(r"<.+?(?:\+0x([0-9a-f]+))?>", note)
            out[name].append((int(note.split(":")[0], 16), op, operands.strip(), start + int(to.group(1) or "0", 16) if to else None))
    return {n: code for n, code in out.items() if any(op.startswith("v_mfma") for _, op, _, _ in code)}


def vector_registers(operands):
    regs = set()
    for a, b, single in re.findall(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)", operands):
        regs.update([int(single)] if single else range(int(a), int(b) + 1))
    return regs


def too_early(code):
    """The instructions that touch a product's result before it has settled on some path.  State: register -> wait states that are left."""
    at = {address: i for i, (address, _, _, _) in enumerate(code)}
    seen, found, todo = [None] * len(code), set(), [(0, {})]
    while todo:
        i, left = todo.pop()
        while i < len(code):
            if seen[i] is not None:
                if all(seen[i].get(r, 0) >= n for r, n in left.items()):
                    break
                left = {r: max(left.get(r, 0), seen[i].get(r, 0)) for r in {*left, *seen[i]}}
            seen[i] = left
            address, op, operands, target = code[i]
            product = op.startswith("v_mfma")
            if not product and re.match("v_|ds_|global_|buffer_|flat_|scratch_", op) and left and vector_registers(operands) & left.keys():
                found.add(f"{address:x}: {op} {operands}")
            step = int(operands, 0) + 1 if op == "s_nop" else 1
            left = {r: n - step for r, n in left.items() if n > step}
            if product:
                left.update(dict.fromkeys(vector_registers(operands.split(",")[0]), NEED[op]))
            if op.startswith("s_cbranch"):
                todo.append((at[target], left))
            if op == "s_endpgm":
                break
            i = at[target] if op == "s_branch" else i + 1
    return found


def test_a_result_read_too_early_is_found():
    def code(*text):
        lines = [f"{4 * i:016x} <f>:" if i == 0 else f"\t{t} // {4 * i:012X}: 0{' <f+0x%x>' % (4 * len(text)) if 'branch' in t else ''}" for i, t in enumerate(("", *text))]
        return functions("\n".join(lines))["f"]
    product, read = "v_mfma_f32_32x32x16_bf16 v[0:15], v[20:23], v[24:27], v[0:15]", "v_max_f32_e32 v40, v3, v3"
    assert too_early(code(product, "s_nop 10", read, "s_endpgm"))
    assert not too_early(code(product, "s_nop 11", read, "s_endpgm"))
    assert too_early(code(product, "s_cbranch_vccz 2", "s_nop 15", "v_mov_b32_e32 v9, v50"))      # around the wait states
    assert not too_early(code(product, "v_mfma_f32_16x16x32_bf16 v[16:19], v[0:3], v[24:27], v[16:19]", "s_nop 10", read, "s_endpgm"))


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs the ROCm disassembler")
def test_every_product_has_settled_before_it_is_read(tmp_path):
    lib = shutil.copy(hb.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    kernels = 0
    for f in sorted(glob.glob(f"{tmp_path}/*gfx950")):
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], check=True, capture_output=True, text=True).stdout
        for name, code in functions(listing).items():
            kernels += 1
            assert not too_early(code), name
    assert kernels > 50
