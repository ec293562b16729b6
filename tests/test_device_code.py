"""What the compiler does not check inside assembler text: wait states around hand-written instructions, looked up in the
disassembly of the library's own gfx950 code."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2211_16270_amd import build as Bld

OBJDUMP = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(Bld.HIPCC))), "llvm", "bin", "llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name of each device function -> its instructions, as (mnemonic, operands) in program order"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    tmp = tmp_path_factory.mktemp("code")
    lib = shutil.copy(Bld.LIB_PATH, tmp)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, cwd=tmp, capture_output=True)
    out, name = {}, None
    for obj in sorted(glob.glob(os.path.join(tmp, "*gfx950*"))):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", obj], check=True, capture_output=True,
                              text=True).stdout
        for line in text.splitlines():
            head = re.match(r"(?:[0-9a-f]+ )?<(.+)>:$", line)
            if head:
                name = head.group(1)
                out[name] = []
            elif name and line.startswith("\t"):
                words = line.split("//")[0].split(None, 1)
                out[name].append((words[0], words[1].strip() if len(words) > 1 else ""))
    assert any("k_scores" in k for k in out) and any("k_lattice_wave" in k for k in out)
    return out


def test_a_wait_state_between_a_write_of_m0_and_a_load_to_lds(kernels):
    copies, close = 0, []
    for name, code in kernels.items():
        for (op, args), (op2, _) in zip(code, code[1:]):
            if not re.search(r"load_lds|lds_addtid", op2):
                continue
            copies += 1
            if op.startswith("s_") and re.match(r"m0\b", args):
                close.append((name, op, op2))
    assert copies > 100
    assert not close, (len(close), close[:3])
