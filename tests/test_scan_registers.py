"""The scan's matrix instructions are written as assembly that updates accumulators in place, so the compiler does not add the
wait states that another instruction would need before it touches one.  Checked in the code it makes: between such an
instruction and the settling wait nothing but matrix instructions names an accumulator's register."""
import os
import re
import subprocess

from paper_2603_10846_amd import binding


def _registers(operands):
    out = set()
    for kind, lo, hi, one_kind, one in re.findall(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", operands):
        out |= {(kind, i) for i in range(int(lo), int(hi) + 1)} if kind else {(one_kind, int(one))}
    return out


def test_nothing_touches_an_accumulator_in_flight(tmp_path):
    out = tmp_path / "evomem.s"
    flags = [f for f in binding.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call(["hipcc", *flags, "--cuda-device-only", "-S", "-o", str(out), binding.SRC], stderr=subprocess.DEVNULL)
    kernels = re.findall(r"^(_ZN3evk11k_scan_mfma\w+):(.*?)s_endpgm", out.read_text(), re.S | re.M)
    assert len(kernels) == 36
    for name, body in kernels:
        accumulators, lines, in_asm = set(), [], False
        for line in map(str.strip, body.splitlines()):
            if line.startswith(";;#ASMSTART") or line.startswith(";APP"):
                in_asm = True
            elif line.startswith(";;#ASMEND") or line.startswith(";NO_APP"):
                in_asm = False
            elif line and line[0] not in ";.":
                lines.append((in_asm, *(line.split(None, 1) + [""])[:2]))
        for asm, op, operands in lines:
            if asm and op.startswith("v_mfma"):
                accumulators |= _registers(operands.split(",")[0])
        assert len(accumulators) in (32, 64, 128), name
        flying = False
        for asm, op, operands in lines:
            if op == "s_nop" and operands == "15":
                flying = False
            elif op.startswith("v_mfma"):
                flying = flying or asm
            elif flying:
                assert not _registers(operands) & accumulators, f"{name}: {op} {operands}"
    os.remove(out)
