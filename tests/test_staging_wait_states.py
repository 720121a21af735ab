"""The large-row GEMM's staging loads are inline assembly, in which the compiler
counts no wait states.  A memory instruction must come at least five wait
states after a vector instruction that writes a scalar register which it reads,
so each load brings them along: whatever the register allocation puts in front
of the block, five wait states of it lie before the load (CPU: the listing of
the built code)."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
WAIT_STATES = 5  # vector write of a scalar register, then a memory read of it


def _listing(tmp_path):
    from paper_2607_12287_amd import build as hip_build

    obj = shutil.copy(hip_build.objects(["k_gemm_tiled.hip"])[0], tmp_path)
    subprocess.check_call([OBJDUMP, "--offloading", os.path.basename(obj)], cwd=tmp_path, stdout=subprocess.DEVNULL)
    code = [f for f in os.listdir(tmp_path) if f.endswith(hip_build.ARCH)]
    assert len(code) == 1, code
    out = subprocess.check_output([OBJDUMP, "-d", "--no-show-raw-insn", code[0]], cwd=tmp_path, text=True)
    return [line.split("//")[0].strip() for line in out.splitlines()]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not installed")
def test_every_staging_load_brings_its_wait_states(tmp_path):
    lines = _listing(tmp_path)
    loads = [i for i, line in enumerate(lines) if re.match(r"buffer_load_dwordx4 .* lds$", line)]
    assert len(loads) >= 100
    for i in loads:
        # the block: the LDS address and the offset by the scalar unit, then the wait
        offset = re.search(r", (s\d+) offen lds$", lines[i]).group(1)
        nop = re.match(r"s_nop (\d+)$", lines[i - 1])
        assert nop, lines[i - 3:i + 1]
        assert lines[i - 2].startswith(f"s_add_u32 {offset}, "), lines[i - 3:i + 1]
        assert lines[i - 3].startswith("s_add_u32 m0, "), lines[i - 3:i + 1]
        assert int(nop.group(1)) + 1 + 2 >= WAIT_STATES
