"""Check of the compiled fused kernels: wait states before broadcast operands.

The green update reads the Khat coefficients with a row broadcast inside an asm
statement (``fmac_bcast`` of ``csrc/solve_kernel.hpp``).  The hardware needs two
wait states between a vector instruction that writes a register and a DPP read
of it (five after a vector instruction that writes EXEC), and the compiler
inserts none for an asm operand: a register copy placed right before its use
would give wrong coefficients without an error.  The coefficients come straight
from LDS reads, so there is no such copy unless the register allocator makes
one; this check of each object's own disassembly shows that it made none.
"""
from __future__ import annotations

import os
import re
import subprocess
import tempfile

LLVM = os.environ.get("STP_LLVM_BIN", "/opt/rocm/llvm/bin")
_LINE = re.compile(r"^\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):(?:.*<\S+?(?:\+0x([0-9a-f]+))?>)?")
_HEAD = re.compile(r"^([0-9a-f]+) <\S+>:$")
_REG = re.compile(r"^(?:-|\|)?v(?:\[(\d+):(\d+)\]|(\d+))")
_DPP_WAIT, _EXEC_WAIT = 2, 5


def disassemble(obj: str, arch: str) -> str:
    """Disassembly of the device code of a HIP object built here."""
    with tempfile.TemporaryDirectory() as d:
        fat, code = os.path.join(d, "fat"), os.path.join(d, "code")
        run = lambda *a: subprocess.run([os.path.join(LLVM, a[0]), *a[1:]], check=True, capture_output=True, text=True)  # noqa: E731
        run("llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", obj, os.devnull)
        run("clang-offload-bundler", "--unbundle", "--type=o", f"--targets=hipv4-amdgcn-amd-amdhsa--{arch}",
            f"--input={fat}", f"--output={code}")
        return run("llvm-objdump", "-d", code).stdout


def _registers(operand: str) -> set:
    m = _REG.match(operand)
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def hazards(listing: str):
    """(broadcast multiply-adds, [those that a write of their operand or of
    EXEC reaches too soon, over every path of branches])."""
    ops = []          # (mnemonic, operands, address, branch target or None)
    base = 0
    for line in listing.splitlines():
        h = _HEAD.match(line)
        if h:
            base = int(h[1], 16)
            continue
        m = _LINE.match(line)
        if m:
            target = base + int(m[4] or "0", 16) if m[1].startswith(("s_cbranch", "s_branch")) else None
            ops.append((m[1], [o.strip() for o in m[2].split(",")], int(m[3], 16), target))
    at = {o[2]: i for i, o in enumerate(ops)}
    count, bad = 0, []
    before = [[] for _ in ops]  # the instructions that can come right before each
    for i, (name, args, addr, target) in enumerate(ops):
        if i + 1 < len(ops) and name not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            before[i + 1].append(i)
        if name == "s_setpc_b64":  # a long branch: s_getpc, s_add_u32 of the distance, s_addc, s_setpc
            get, add = ops[i - 3], ops[i - 2]
            if get[0] == "s_getpc_b64" and add[0] == "s_add_u32":
                distance = int(add[1][2], 0)
                distance -= (distance & 0x80000000) << 1 if distance > 0 else 0
                target = get[2] + 4 + distance
            if target not in at:
                bad.append(f"{addr:x}: branch to an unknown place")
        if target in at:
            before[at[target]].append(i)
    for i, (name, args, addr, _) in enumerate(ops):
        if not (name.startswith("v_fmac") and "row_newbcast" in " ".join(args)):
            continue
        count += 1
        source = _registers(args[1])
        todo, seen = [(j, 0) for j in before[i]], set()
        while todo:
            j, waited = todo.pop()
            if (j, waited) in seen or waited >= _EXEC_WAIT:
                continue
            seen.add((j, waited))
            pname, pargs = ops[j][0], ops[j][1]
            if pname.startswith("v_"):
                written = _registers(pargs[0]) | (_registers(pargs[1]) if "swap" in pname else set())
                if (waited < _DPP_WAIT and written & source) or pname.startswith("v_cmpx"):
                    bad.append(f"{addr:x}: {name} {', '.join(args)} after {ops[j][2]:x}: {pname} {', '.join(pargs)}")
                    break
            wait = int(pargs[0], 0) + 1 if pname == "s_nop" else 1
            todo += [(k, waited + wait) for k in before[j]]
    return count, bad


def check(obj: str, arch: str) -> int:
    """Raises if a broadcast of `obj` could read too soon; returns their number."""
    count, bad = hazards(disassemble(obj, arch))
    if bad:
        raise RuntimeError(f"{os.path.basename(obj)}: {len(bad)} broadcast(s) too close to a write:\n" + "\n".join(bad[:10]))
    return count
