"""The scan's matrix instructions are written as assembly that updates accumulators in place, so the compiler does not add the
wait states that another instruction would need before it touches one.  Checked in the code it makes: between such an
instruction and the settling wait nothing but matrix instructions names an accumulator's register; and no vector instruction
writes an operand of one in the two wait states before it.
Query blocks go straight to LDS by assembly too, which sets M0 and counts on the order of the loads.  Checked: no value that the
compiler put into M0 is used behind such a load, and enough loads follow the last of a step's before the wait that lets them through.
Where operands pass through rings (16-bit stores, 128 or 256 queries to a tile) the waits count on how many loads follow, each group of wavefronts
for itself.  Checked: the k-loop has the reads, loads, waits and barriers that its schedule rests on, in their order, and no other memory
operation and no other wait for one."""
import os
import re
import subprocess

from paper_2603_10846_amd import binding


def _registers(operands):
    out = set()
    for kind, lo, hi, one_kind, one in re.findall(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", operands):
        out |= {(kind, i) for i in range(int(lo), int(hi) + 1)} if kind else {(one_kind, int(one))}
    return out


def _memory_events(body):
    """Runs of: r LDS reads, L loads to LDS, g other memory operations, M matrix instructions; Wn waits for memory, B barriers (behind a wait for all LDS
    reads)."""
    events, reads_pending = [], False
    for line in map(str.strip, body.splitlines()):
        if not line or line[0] in ";.":
            continue
        op = line.split()[0]
        if op.startswith("global_load_lds"):
            e = "L"
        elif op.startswith(("global_", "buffer_", "scratch_", "flat_")):
            e = "g"
        elif op.startswith("v_mfma"):
            e = "M"
        elif op.startswith("ds_read"):
            e, reads_pending = "r", True
        elif op == "s_barrier":
            e = "B?" if reads_pending else "B"
        elif op == "s_waitcnt":
            if "lgkmcnt(0)" in line:
                reads_pending = False
            vm = re.search(r"vmcnt\((\d+)\)", line)
            if not vm:
                continue
            e = f"W{vm.group(1)}"
        else:
            continue
        if events and events[-1][0] == e and e in "rLgM":
            events[-1][1] += 1
        else:
            events.append([e, 1])
    return " ".join(e if n == 1 else f"{e}x{n}" for e, n in events)


def test_nothing_touches_an_accumulator_in_flight(tmp_path):
    out = tmp_path / "evomem.s"
    flags = [f for f in binding.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call(["hipcc", *flags, "--cuda-device-only", "-S", "-o", str(out), binding.SRC], stderr=subprocess.DEVNULL)
    kernels = re.findall(r"^(_ZN3evk11k_scan_mfma\w+):(.*?)s_endpgm", out.read_text(), re.S | re.M)
    assert len(kernels) == 44
    direct = 0
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

        recent = []                                          # what vector instructions wrote in the last two wait states
        for asm, op, operands in lines:
            if asm and op.startswith("v_mfma"):
                read = set().union(*(_registers(x) for x in operands.split(", ")[1:3]))
                assert not any(read & written for written in recent), f"{name}: {op} {operands}"
            states = int(operands) + 1 if op == "s_nop" else 1
            written = _registers(operands.split(",")[0]) if op.startswith("v_") and not op.startswith(("v_mfma", "v_cmp", "v_readlane", "v_readfirstlane")) else set()
            recent = (recent + [set()] * (states - 1) + [written])[-2:]

        theirs = False                                       # what M0 holds is the compiler's
        behind = None                                        # memory operations behind the last load to LDS
        for asm, op, operands in lines:
            if re.search(r"\bm0\b", operands):
                if op.startswith("s_") and operands.startswith("m0"):
                    theirs = not asm
                else:
                    assert not asm and theirs, f"{name}: {op} {operands}"
            if asm and op.startswith("global_load_lds"):
                behind, direct = 0, direct + 1
            elif op.startswith(("global_", "buffer_", "scratch_", "flat_")) and behind is not None:
                behind += 1
            elif asm and op == "s_waitcnt" and behind is not None:
                assert behind >= int(re.fullmatch(r"vmcnt\((\d+)\)", operands).group(1)), f"{name}: {operands} {behind} operations behind the loads"
    assert direct > 0

    rings = 0
    for name, body in kernels:
        dt, mq, wq = map(int, re.match(r"_ZN3evk11k_scan_mfmaILi(\d)ELi(\d)ELi(\d)E", name).groups())
        if dt == 0 or mq * wq < 8:
            continue
        rings += 1
        # Half a query block is 16 * mq * wq fragments' rows of 64 bytes, loaded by four wavefronts, 1 KB at a time; a bank block is 32 KB: eight loads.
        # The query group waits, at the end of half i + 1, until only the loads of half i + 3 are left: q of them.  The bank group waits, in the second
        # half of block m + 1, until only those of block m + 2 are: eight.  At the start two halves and two blocks are asked for.
        q, fetch, multiply = mq * wq // 4, f"rx{mq + 4} Lx{mq * wq // 4 + 4}", f"B Mx{4 * mq} W{mq * wq // 4} B"
        events = _memory_events(body)
        assert events.count(f"Lx{2 * q} W{q} Lx16 W8 B ") == 1, f"{name}: {events}"
        assert events.count(f" B {fetch} {multiply} B {fetch} W8 {multiply} ") == 1, f"{name}: {events}"
        assert events.count("L") == 4, f"{name}: {events}"
    assert rings == 20
    os.remove(out)
