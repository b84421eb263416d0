"""Wait states of the hand-written instructions, read from the disassembly of
the built library (gfx950).

The compiler inserts the wait states that the hardware does not check itself,
but it does not look inside inline assembly.  Three rules of the CDNA ISA
documents ("manually inserted wait states") concern what this library writes
by hand, and `violations` checks them over all paths through each kernel:

  m0     an SALU write of M0 and a load into LDS, which takes its LDS base from
         M0, need one instruction in between
  sgpr   a VALU write of an SGPR (v_readlane, v_readfirstlane, a comparison)
         and a vector-memory instruction that reads it need five
  acc    the result of a matrix instruction in accumulation registers (the
         hand-written products) and anything but another product that adds to
         the same registers need 19; copies and spills that a compiler might
         put between the products show here too
"""
from __future__ import annotations

import glob
import os
import re
import shutil
import subprocess

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
NEED = {"m0": 1, "sgpr": 5, "acc": 19}
_VMEM = ("global_", "buffer_", "scratch_", "flat_")
_REG = re.compile(r"\b([vas])(?:\[(\d+):(\d+)\]|(\d+)\b)")
_LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]{12}):(.*)$")
_TARGET = re.compile(r"<(\S+?)(?:\+0x([0-9a-f]+))?>\s*$")


def disassemble(lib: str, tmp: str) -> list[str]:
    """Listings of the gfx950 code objects inside a shared library."""
    copy = shutil.copy(lib, os.path.join(tmp, "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", copy], check=True, capture_output=True)
    objs = sorted(glob.glob(os.path.join(tmp, "lib.so.*gfx950*")))
    return [subprocess.run([OBJDUMP, "-d", o], check=True, capture_output=True, text=True).stdout for o in objs]


def _regs(text: str) -> frozenset:
    out = set()
    for kind, lo, hi, one in _REG.findall(text):
        out.update((kind, i) for i in range(int(lo or one), int(hi or one) + 1))
    return frozenset(out)


class Instr:
    def __init__(self, op, args, addr):
        self.op, self.args, self.addr = op, args, addr
        ops = [a.strip() for a in args.split(",")] if args else []
        dst = ops[0] if ops else ""
        self.waits = int(ops[0], 0) + 1 if op == "s_nop" else 1
        self.mfma = "mfma" in op
        self.m0_write = op.startswith("s_") and dst == "m0" and not op.startswith("s_cmp")
        self.lds_load = "_load_lds_" in op
        self.vmem = op.startswith(_VMEM)
        self.regs = _regs(args)
        valu = op.startswith("v_") and not self.mfma
        self.sgpr_write = frozenset(r for r in _regs(dst) if r[0] == "s") if valu else frozenset()
        self.acc = frozenset(r for r in _regs(dst) if r[0] == "a") if self.mfma else frozenset()
        # accumulation registers that need the finished result: all but a
        # product's own accumulator (the same registers in and out)
        used = frozenset(r for r in self.regs if r[0] == "a")
        if self.mfma and len(ops) > 3 and ops[3].split()[0] == dst:
            used = frozenset(r for r in _regs(",".join(ops[1:3])) if r[0] == "a")
        self.acc_use = used
        self.preds: list[int] = []


def parse(listing: str) -> dict[str, list[Instr]]:
    """Kernels (by symbol) with their instructions and predecessors."""
    kernels, code, start, targets = {}, None, 0, []
    for line in listing.splitlines():
        head = re.match(r"^([0-9a-f]{16}) <(.+)>:$", line)
        if head:
            code, start = [], int(head[1], 16)
            kernels[head[2]] = code
            continue
        m = _LINE.match(line)
        if code is None or not m:
            continue
        ins = Instr(m[1], m[2], int(m[3], 16))
        if m[1].startswith(("s_cbranch", "s_branch")):
            t = _TARGET.search(m[4])
            ins.target = start + int(t[2] or "0", 16)
        code.append(ins)
    for code in kernels.values():
        at = {i.addr: n for n, i in enumerate(code)}
        for n, i in enumerate(code):
            if i.op not in ("s_branch", "s_endpgm", "s_setpc_b64") and n + 1 < len(code):
                code[n + 1].preds.append(n)
            if hasattr(i, "target") and i.target in at:
                code[at[i.target]].preds.append(n)
    return kernels


def exec_constants(code) -> list[str]:
    """Hand-written writes of EXEC that put a constant there and do not put back
    what they found: the compiler does not see them, so the lanes that it had
    switched off would run on.  Allowed is a copy of EXEC, the constant, and
    the copy back before any branch."""
    out = []
    for n, i in enumerate(code):
        if i.op != "s_mov_b64" or not re.fullmatch(r"exec, 1", i.args):
            continue
        kept = re.fullmatch(r"(s\[\d+:\d+\]), exec", code[n - 1].args) if n else None
        back = next((j for j in code[n + 1:] if j.args.startswith("exec") or j.op.startswith(("s_cbranch", "s_branch"))),
                    None)
        if not (kept and code[n - 1].op == "s_mov_b64" and back and back.args == "exec, " + kept[1]):
            out.append("%s %s" % (i.op, i.args))
    return out


def _before(code, n, states):
    """Instructions that can run fewer than `states` wait states before n."""
    best, todo = {}, [(p, 0) for p in code[n].preds]
    while todo:
        p, w = todo.pop()
        if w >= states or best.get(p, states) <= w:
            continue
        best[p] = w
        yield code[p], w
        todo.extend((q, w + code[p].waits) for q in code[p].preds)


def violations(listing: str) -> list[str]:
    out = []
    for name, code in parse(listing).items():
        for n, i in enumerate(code):
            if i.lds_load:
                out += ["m0: %s: %s %s" % (name, i.op, i.args)
                        for p, _ in _before(code, n, NEED["m0"]) if p.m0_write]
            if i.vmem:
                out += ["sgpr: %s: %s %s after %s %s" % (name, i.op, i.args, p.op, p.args)
                        for p, _ in _before(code, n, NEED["sgpr"]) if p.sgpr_write & i.regs]
            if i.acc_use:
                out += ["acc: %s: %s %s after %s %s" % (name, i.op, i.args, p.op, p.args)
                        for p, _ in _before(code, n, NEED["acc"]) if p.acc & i.acc_use]
    return out
