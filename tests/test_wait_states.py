"""A memory instruction that takes its address from scalar registers comes five wait states or more after a vector instruction
that wrote them (data hazard of the CDNA ISA, not checked by the hardware).  The compiler sees to it around its own loads, but
does not look into inline assembly; so the machine code of the built library is checked as it is."""
import glob
import os
import re
import shutil
import subprocess

import pytest

import paper_2603_04127_amd as dk

OBJDUMP = shutil.which("llvm-objdump", path=os.pathsep.join(["/opt/rocm/llvm/bin", os.environ.get("PATH", "")]))
WAIT_STATES = 5
MEMORY = ("global_", "buffer_", "flat_", "scratch_")
CARRY_OUT = ("v_add_co_", "v_addc_co_", "v_sub_co_", "v_subb_co_", "v_subrev_co_", "v_subbrev_co_", "v_div_scale", "v_mad_u64", "v_mad_i64")


def scalars(operand):
    """Scalar registers that an operand of the listing names."""
    r = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if r:
        return {f"s{i}" for i in range(int(r[1]), int(r[2]) + 1)}
    if re.fullmatch(r"s\d+", operand):
        return {operand}
    return {"vcc": {"vcc_lo", "vcc_hi"}, "vcc_lo": {"vcc_lo"}, "vcc_hi": {"vcc_hi"}}.get(operand, set())


def parse(listing):
    """[(address, mnemonic, operands, address of the branch's target or None)] of a disassembly."""
    code = []
    for line in listing.splitlines():
        r = re.match(r"\s+([a-z]\w+)\s*(.*?)\s*// ([0-9A-F]+):", line)
        if not r:
            continue
        ops = [o.split()[0] for o in r[2].split(",") if o.strip()]
        target = None
        if r[1].startswith(("s_branch", "s_cbranch")):
            off = int(ops[0])
            target = int(r[3], 16) + 4 + 4 * (off - 65536 if off >= 32768 else off)
        code.append((int(r[3], 16), r[1], ops, target))
    return code


def writes(name, ops):
    """Scalar registers that a vector instruction writes."""
    if not name.startswith("v_"):
        return set()
    if name.startswith("v_cmpx"):
        return set()
    w = scalars(ops[0]) if ops else set()
    if len(ops) > 1 and name.startswith(CARRY_OUT):
        w |= scalars(ops[1])
    return w


def violations(code):
    at = {a: i for i, (a, *_) in enumerate(code)}
    jumps = {}
    for i, (_, _, _, target) in enumerate(code):
        if target in at:
            jumps.setdefault(at[target], []).append(i)
    bad, checked = [], 0
    for i, (addr, name, ops, _) in enumerate(code):
        if not name.startswith(MEMORY):
            continue
        need = set().union(*map(scalars, ops)) if ops else set()
        if not need:
            continue
        checked += 1
        todo, seen = [(i, 0)], {}
        while todo:
            j, states = todo.pop()
            before = list(jumps.get(j, []))
            if j > 0 and code[j - 1][1] not in ("s_branch", "s_endpgm", "s_setpc_b64"):
                before.append(j - 1)
            for k in before:
                _, kn, ko, _ = code[k]
                if writes(kn, ko) & need:
                    bad.append((hex(addr), name, f"{states} wait states after", hex(code[k][0]), kn))
                    continue
                n = states + (int(ko[0], 0) + 1 if kn == "s_nop" else 1)
                if n < WAIT_STATES and seen.get(k, WAIT_STATES) > n:
                    seen[k] = n
                    todo.append((k, n))
    return bad, checked


def test_the_check_sees_the_hazard():
    listing = """
\tv_readfirstlane_b32 s4, v3 // 000000000000: 00
\ts_mov_b32 m0, s6 // 000000000004: 00
\ts_nop {n} // 000000000008: 00
\tglobal_load_lds_dwordx4 v2, s[4:5] // 00000000000C: 00
"""
    assert violations(parse(listing.format(n=2))) == ([("0xc", "global_load_lds_dwordx4", "4 wait states after", "0x0", "v_readfirstlane_b32")], 1)
    assert violations(parse(listing.format(n=3))) == ([], 1)


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_scalar_addresses_of_the_library(tmp_path):
    dk.lib()
    so = tmp_path / "lib.so"
    shutil.copy(os.path.join(os.path.dirname(dk.__file__), "libdark.so"), so)
    subprocess.check_call([OBJDUMP, "--offloading", str(so)], stdout=subprocess.DEVNULL, cwd=tmp_path)
    total, bad = 0, []
    for obj in glob.glob(str(tmp_path / "*gfx950*")):
        b, n = violations(parse(subprocess.check_output([OBJDUMP, "-d", obj], text=True)))
        total += n
        bad += b
    assert total > 500
    assert not bad, bad[:10]
