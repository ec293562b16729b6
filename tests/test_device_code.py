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


def _registers(args):
    """the vector registers each operand of an instruction names, as sets of ('v' | 'a', number)"""
    out = []
    for a in args.split(","):
        m = re.match(r"\s*([va])(?:(\d+)|\[(\d+):(\d+)\])", a)
        lo, hi = (int(m.group(2) or m.group(3)), int(m.group(2) or m.group(4))) if m else (0, -1)
        out.append({(m.group(1), i) for i in range(lo, hi + 1)} if m else set())
    return out


def _valu(op):
    return op.startswith("v_") and not op.startswith("v_mfma")


def test_wait_states_around_matrix_instructions(kernels):
    # per pass of a matrix instruction one wait state; a 32x32x16 bf16 product has eight passes and its result may be touched by a
    # vector instruction eleven states later; a vector instruction that writes an operand stands two states ahead
    BEFORE, DEPTH, AFTER = 2, 8, 11
    seen, bad = 0, []
    for name, code in kernels.items():
        if "k_scores" not in name:
            continue
        parsed = [(op, args, _registers(args) if op.startswith("v_") else []) for op, args in code]
        for at, (op, args, regs) in enumerate(parsed):
            if not op.startswith("v_mfma_f32_32x32x16_bf16"):
                continue
            seen += 1
            operands = regs[1] | regs[2] | regs[3]
            states = 0
            for op2, args2, regs2 in reversed(parsed[max(0, at - BEFORE):at]):
                if states >= BEFORE or op2.startswith("v_mfma"):
                    break
                written = regs2[0] | (regs2[1] if "swap" in op2 else set()) if _valu(op2) else set()
                if written & operands:
                    bad.append((name, "written too late", op2, args2, args))
                states += 1 + (int(args2, 0) if op2 == "s_nop" else 0)
            states = 0
            for op2, args2, regs2 in parsed[at + 1:]:
                if states >= AFTER or op2 in ("s_branch", "s_endpgm"):
                    break
                if _valu(op2) and regs[0] & set().union(*regs2):
                    bad.append((name, "touched too early", op2, args2, args))
                # (the next matrix instruction leaves when this one's passes are through)
                states += DEPTH if op2.startswith("v_mfma") else 1 + (int(args2, 0) if op2 == "s_nop" else 0)
    assert seen > 2000
    assert not bad, (len(bad), bad[:3])
