"""The listing of the built attention kernels (CPU): the first operand of every
matrix product is a key or value fragment, so each of its registers was last
written by a load, or by the zeroing of padding and of keys past the stream's
end, and by nothing in between.  (The compiler once gave registers of a value
fragment to the softmax before its last product; fp32 models with heads wider
than 64 then returned wrong rows.)"""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
KEEP = ("v_cndmask_b32", "v_and_b32", "v_accvgpr")  # zeroing, or a move between the register files


def _registers(operand):
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]", operand)
    if m:
        return [f"{m.group(1)}{i}" for i in range(int(m.group(2)), int(m.group(3)) + 1)]
    return [operand] if re.fullmatch(r"[va]\d+", operand) else []


def _overwritten(lines):
    """(kernels, products, [(kernel, product, register, writer)])"""
    kernel, wrote, found, kernels, products = None, {}, [], 0, 0
    for line in lines:
        m = re.match(r"[0-9a-f]+ <(\S+)>:$", line)
        if m:
            kernel, wrote = ("attn_kernel" in m.group(1) and m.group(1)), {}
            kernels += bool(kernel)
            continue
        m = re.match(r"(v_\S+|ds_read\S*|global_load\S*|buffer_load\S*)\s+(.*)$", line)
        if not kernel or not m:
            continue
        op, args = m.group(1), [a.split(" ")[0] for a in re.split(r",\s*(?![^\[]*\])", m.group(2))]
        if op.startswith("v_mfma"):
            products += 1
            found += [(kernel, line, r, wrote[r]) for r in _registers(args[1]) if wrote.get(r, "load") != "load"]
        if op.startswith("v_cmp"):
            continue
        loads = op.startswith(("global_load", "buffer_load", *KEEP)) or (
            op.startswith("v_mov_b32") and (not _registers(args[1]) or wrote.get(args[1]) == "load"))
        for r in _registers(args[0]) + (_registers(args[1]) if "swap" in op else []):
            wrote[r] = "load" if loads else op
    return kernels, products, found


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not installed")
def test_key_and_value_fragments_reach_their_products(tmp_path):
    from paper_2607_12287_amd import build as hip_build

    obj = shutil.copy(hip_build.objects(["k_attn.hip"])[0], tmp_path)
    subprocess.check_call([OBJDUMP, "--offloading", os.path.basename(obj)], cwd=tmp_path, stdout=subprocess.DEVNULL)
    code = [f for f in os.listdir(tmp_path) if f.endswith(hip_build.ARCH)]
    assert len(code) == 1, code
    out = subprocess.check_output([OBJDUMP, "-d", "--no-show-raw-insn", code[0]], cwd=tmp_path, text=True)
    kernels, products, found = _overwritten([line.split("//")[0].strip() for line in out.splitlines()])
    assert kernels >= 45 and products >= 45 * 3, (kernels, products)
    assert not found, found[:4]
