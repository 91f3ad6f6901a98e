"""The direct-to-LDS copies are inline assembly, so the compiler does not put the
hardware's wait states between them and what writes their scalar operands.
Checked on the instructions of the built library: five wait states from a VALU
write of the base address (a spilled scalar register's reload is one) or of M0
to the copy, one from a scalar write of M0.  A copy too soon after such a write
reads a stale address."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_07740_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _scalars(operand):
    """Scalar registers named by an operand."""
    m = re.match(r"s\[(\d+):(\d+)\]$", operand)
    if m:
        return {"s%d" % i for i in range(int(m[1]), int(m[2]) + 1)}
    if operand == "vcc":
        return {"vcc_lo", "vcc_hi"}
    return {operand} if re.match(r"(s\d+|m0|vcc_lo|vcc_hi)$", operand) else set()


def find_short_waits(listing):
    """(kernel, instruction, register, wait states) of each copy too soon after a write."""
    found, copies = [], 0
    kernel, pos, valu, salu_m0 = None, 0, {}, -10
    for line in listing.split("\n"):
        m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if m:
            kernel, valu, salu_m0 = m[1], {}, -10
            continue
        ins = line.split("//")[0].strip()
        if not line.startswith("\t") or not ins:
            continue
        op, _, rest = ins.partition(" ")
        args = [a.split()[0] for a in rest.split(",") if a.split()]
        if op == "s_nop":
            pos += int(args[0], 0) + 1
            continue
        if "_lds_" in op:
            copies += 1
            for r in set().union(*map(_scalars, args)) | {"m0"}:
                if pos - valu.get(r, -10) - 1 < 5:
                    found.append((kernel, ins, r, pos - valu[r] - 1))
            if pos - salu_m0 - 1 < 1:
                found.append((kernel, ins, "m0", pos - salu_m0 - 1))
        elif op.startswith("v_"):  # the last writer of a scalar register is a VALU instruction
            dst = set(_scalars(args[0])) if args else set()
            if len(args) > 1 and ("_co_" in op or "div_scale" in op or op.startswith("v_mad_")):
                dst |= _scalars(args[1])
            for r in dst:
                valu[r] = pos
                if r == "m0":
                    salu_m0 = -10
        elif op.startswith("s_") and args and not op.startswith(("s_cmp", "s_bitcmp", "s_cbranch")):
            for r in _scalars(args[0]):
                valu.pop(r, None)
                if r == "m0":
                    salu_m0 = pos
        pos += 1
    return found, copies


def test_scan_sees_a_short_wait():
    bad = ("0 <k>:\n\tv_readlane_b32 s4, v1, 2  // 0\n\tv_readlane_b32 s5, v1, 3  // 0\n"
           "\ts_mov_b32 m0, s9  // 0\n\ts_nop 0  // 0\n\tglobal_load_lds_dwordx4 v2, s[4:5]  // 0\n")
    found, copies = find_short_waits(bad)
    assert copies == 1 and {f[2:] for f in found} == {("s4", 3), ("s5", 2)}
    good = bad.replace("s_nop 0", "s_mov_b64 vcc, s[4:5]").replace("v2, s[4:5]", "v2, vcc")
    assert find_short_waits(good) == ([], 1)
    found, _ = find_short_waits("0 <k>:\n\ts_mov_b32 m0, s9  // 0\n"
                                "\tglobal_load_lds_dwordx4 v2, s[4:5]  // 0\n")
    assert [f[2:] for f in found] == [("m0", 0)]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler in this installation")
def test_copies_keep_their_wait_states(tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    lib = shutil.copy(build.LIB, str(tmp_path / "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=str(tmp_path), check=True,
                   capture_output=True, timeout=120)
    objs = sorted(p for p in os.listdir(str(tmp_path)) if p.endswith("gfx950"))
    assert objs
    total = 0
    for o in objs:
        text = subprocess.run([OBJDUMP, "-d", o], cwd=str(tmp_path), check=True,
                              capture_output=True, text=True, timeout=120).stdout
        found, copies = find_short_waits(text)
        assert not found, found[:4]
        total += copies
    assert total > 100  # the prefill and decode kernels' copies were seen
