"""Wait states around the memory instructions that the kernels issue from inline assembly, looked up in the built library's own code.

A vector memory instruction reads a scalar register five wait states after a vector instruction (v_readfirstlane, v_readlane of a
spilled register) wrote it at the earliest.  The compiler sees to that for its own instructions and not inside an asm statement, so
where a pointer is made, or a register spilled, decides whether it holds.
"""
import os
import re
import shutil
import subprocess
from collections import defaultdict

import pytest

OBJDUMP = shutil.which("llvm-objdump", path=os.pathsep.join(["/opt/rocm/llvm/bin", os.environ.get("PATH", "")]))
LOAD, STATES = "global_load_lds_dwordx4", 5


def scalar_registers(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", operand)
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def functions(listing):
    """(name, [(opcode, operands, index of the branch target or None), ...]) of every function of a disassembly."""
    name, start, code = None, 0, []

    def resolved():
        at = {address: i for i, (address, *_) in enumerate(code)}
        return name, [(op, args, at.get(target)) for _, op, args, target in code]

    for line in listing.splitlines():
        head = re.match(r"([0-9a-f]{16}) <(.*)>:", line)
        if head:
            if name:
                yield resolved()
            name, start, code = head[2], int(head[1], 16), []
            continue
        m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):(.*)", line)
        if m:
            target = re.search(r"<[^>]*?(?:\+0x([0-9a-f]+))?>\s*$", m[4]) if m[1].startswith(("s_cbranch", "s_branch")) else None
            code.append((int(m[3], 16), m[1], [x.strip() for x in m[2].split(",")] if m[2] else [],
                         start + int(target[1] or "0", 16) if target else None))
    if name:
        yield resolved()


def states_before(code, index, before):
    """Wait states between the load at `index` and the nearest vector write of its base on any way to it, at most STATES."""
    base = scalar_registers(code[index][1][1])
    best, seen, todo = STATES, {}, [(p, 0) for p in before[index]]
    while todo:
        p, waited = todo.pop()
        if waited >= best or seen.get(p, STATES) <= waited:
            continue
        seen[p] = waited
        op, args, _ = code[p]
        if op.startswith("v_") and any(scalar_registers(a) & base for a in args[:2 if "_co_" in op else 1]):
            best = waited
            continue
        if op.startswith("s_") and args and base <= scalar_registers(args[0]):
            continue                                          # a scalar instruction waits for the vector one by itself
        todo += [(q, waited + (int(args[0], 0) + 1 if op == "s_nop" else 1)) for q in before[p]]
    return best


def listings(tmp_path):
    """The disassembly of every code object of the built library."""
    lib = tmp_path / "lib.so"
    shutil.copy(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_28115_amd", "libcivic.so"), lib)
    subprocess.run([OBJDUMP, "--offloading", lib.name], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    for obj in sorted(tmp_path.glob("*gfx950*")):
        yield subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(obj)], check=True, stdout=subprocess.PIPE, text=True).stdout


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_loads_into_lds_wait_for_their_base(tmp_path):
    loads = 0
    for listing in listings(tmp_path):
        if LOAD not in listing:
            continue
        for name, code in functions(listing):
            before = defaultdict(list)
            for i, (op, _, target) in enumerate(code):
                if target is not None:
                    before[target].append(i)
                if op not in ("s_branch", "s_endpgm", "s_setpc_b64") and i + 1 < len(code):
                    before[i + 1].append(i)
            for i, (op, _, _) in enumerate(code):
                if op == LOAD:
                    loads += 1
                    assert states_before(code, i, before) >= STATES, (name, i)
    assert loads > 100                                        # the listings were read


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_written_through_stores_keep_their_data_for_a_state(tmp_path):
    """A store of more than 8 bytes reads its data a wait state after it was issued; those written in assembly wait it out themselves."""
    stores = 0
    for listing in listings(tmp_path):
        for name, code in functions(listing) if "sc1" in listing else ():
            for (op, args, _), (after, _, _) in zip(code, code[1:]):
                if op == "global_store_dwordx4" and any("sc1" in a for a in args):
                    stores += 1
                    assert after == "s_nop", name
    assert stores >= 10                                       # the merged rows
