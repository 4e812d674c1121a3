"""Wait states that the hardware does not insert and that the compiler does not see inside inline assembly, checked on the
instructions of the built library:
- a load from memory straight into LDS reads M0 (its LDS address); between a scalar write of M0 and the load there has to be one
  wait state, or the load may take the M0 before it;
- a memory instruction that reads a scalar register needs five wait states after a vector instruction that wrote it."""
import os
import re
import subprocess

import pytest

import paper_2203_15980_amd as dl

OBJDUMP = "/opt/rocm/lib/llvm/bin/llvm-objdump"


def _programs(tmp):
    """The library's device code, one list of (mnemonic, operands) per code object."""
    lib = os.path.join(os.path.dirname(os.path.abspath(dl.__file__)), "libdelta.so")
    link = os.path.join(tmp, "lib.so")
    os.symlink(lib, link)
    subprocess.run([OBJDUMP, "--offloading", link], cwd=tmp, check=True, stdout=subprocess.DEVNULL)
    for name in sorted(os.listdir(tmp)):
        if "gfx950" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(tmp, name)], check=True, stdout=subprocess.PIPE).stdout.decode()
        code = [line.split("//")[0].split(None, 1) for line in text.splitlines() if line.startswith("\t")]
        yield [(c[0], c[1].strip() if len(c) > 1 else "") for c in code if c]


def _scalars(operand):
    """Numbers of the scalar registers an operand names."""
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand) or re.fullmatch(r"s(\d+)()", operand)
    return set(range(int(m.group(1)), int(m.group(2) or m.group(1)) + 1)) if m else set()


def _wait_states(op, args):
    return int(args, 0) + 1 if op == "s_nop" else 1


def hazards(code):
    """(loads into LDS seen, descriptions of those issued too early)."""
    loads, bad = 0, []
    for i, (op, args) in enumerate(code):
        operands = [a.strip() for a in args.replace(" lds", ", lds").split(",")]
        if not ("load_lds" in op or (op.startswith("buffer_load") and operands[-1] == "lds")):
            continue
        loads += 1
        reads = set().union(*[_scalars(a.split()[0]) for a in operands if a])
        states = 0
        for before, what in reversed(code[max(0, i - 5):i]):
            target = what.split(",")[0].strip()
            if states < 1 and target == "m0" and before.startswith("s_"):
                bad.append("%s %s directly after %s %s" % (op, args, before, what))
            if states < 5 and before.startswith("v_") and _scalars(target) & reads:
                bad.append("%s %s: %d wait states after %s %s" % (op, args, states, before, what))
            states += _wait_states(before, what)
    return loads, bad


def test_the_check_itself():
    load = ("global_load_lds_dwordx4", "v8, s[10:11]")
    assert hazards([("s_mov_b32", "m0, s20"), load]) == (1, ["global_load_lds_dwordx4 v8, s[10:11] directly after s_mov_b32 m0, s20"])
    assert hazards([("s_mov_b32", "m0, s20"), ("s_nop", "0"), load]) == (1, [])
    assert len(hazards([("v_readfirstlane_b32", "s11, v1"), ("s_mov_b32", "m0, s20"), ("s_nop", "0"), load])[1]) == 1
    assert hazards([("v_readfirstlane_b32", "s11, v1"), ("s_mov_b32", "m0, s20"), ("s_nop", "3"), load]) == (1, [])


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_loads_into_lds_wait_for_their_address(tmp_path):
    loads, bad = 0, []
    for code in _programs(str(tmp_path)):
        n, b = hazards(code)
        loads += n
        bad += b
    assert loads > 0 and not bad, "%d of %d, first: %s" % (len(bad), loads, bad[0])
