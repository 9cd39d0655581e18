"""Order of matrix products in the compiled kernels.

On gfx950 a matrix product that takes its accumulator straight from a product of another
operand format (FP8 against FP16) gives other bits than with something in between, and the
compiler does not keep the two apart: measured on 5e5 values, an FP16 product right behind the
FP8 product on one accumulator changes half of them, with the product of another accumulator
or a wait of 16 states in between none.  The order in the source does not bind the compiler
(a rewording that kept it put such products next to each other), so the build reads the order
from the kernels it has compiled and refuses a library that holds such a pair.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import tempfile

WAIT = 16  # wait states that keep two formats apart

_FUNC = re.compile(r"^([0-9a-f]+) <(.*)>:$")
_ADDR = re.compile(r"// ([0-9A-F]+):")
_TARGET = re.compile(r"<.*\+0x([0-9a-f]+)>$")
_REGS = re.compile(r"([av])\[(\d+):(\d+)\]")


def _tool(name: str) -> str:
    clang = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    for d in ("/opt/rocm/llvm/bin", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(clang))), "llvm", "bin")):
        if os.path.exists(os.path.join(d, name)):
            return os.path.join(d, name)
    raise RuntimeError("%s not found" % name)


def disassemble(obj: str) -> str:
    """Assembly text of the gfx950 code in a host object file."""
    with tempfile.TemporaryDirectory() as d:
        fat, code = os.path.join(d, "fat"), os.path.join(d, "code")
        subprocess.run([_tool("llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat, obj, os.path.join(d, "o")],
                       check=True, capture_output=True)
        subprocess.run([_tool("clang-offload-bundler"), "--type=o", "--unbundle",
                        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + fat, "--output=" + code],
                       check=True, capture_output=True)
        r = subprocess.run([_tool("llvm-objdump"), "-d", "--no-show-raw-insn", code], check=True, capture_output=True,
                           text=True)
        return r.stdout


def _format(op: str) -> str:
    return op.split("_", 4)[-1] if op.startswith("v_mfma_") else ""


def _functions(text: str):
    """(name, [(offset, opcode, operands, branch target or None)]) of each function."""
    name, base, body = None, 0, []
    for line in text.splitlines():
        m = _FUNC.match(line)
        if m:
            if name:
                yield name, body
            name, base, body = m.group(2), int(m.group(1), 16), []
            continue
        a = _ADDR.search(line)
        if not a or not name:
            continue
        ins = line[:a.start()].split(None, 1)
        t = _TARGET.search(line) if "branch" in ins[0] else None
        body.append((int(a.group(1), 16) - base, ins[0], ins[1].strip() if len(ins) > 1 else "",
                     int(t.group(1), 16) if t else None))
    if name:
        yield name, body


def adjacent_formats(text: str) -> list:
    """[(function, offset, opcode)] of products that follow one of another format on their
    accumulator with no product and fewer than WAIT states in between, on any path."""
    found = []
    for name, body in _functions(text):
        if len({_format(op) for _, op, _, _ in body if op.startswith("v_mfma_")}) < 2:
            continue
        at = {off: i for i, (off, _, _, _) in enumerate(body)}
        # reached[i]: states before instruction i, (format, first, last register, waits since)
        reached = [set() for _ in body]
        bad = set()
        work = [(0, None)]
        while work:
            i, st = work.pop()
            while i < len(body):
                if st in reached[i]:
                    break
                reached[i].add(st)
                off, op, args, target = body[i]
                if op.startswith("v_mfma_"):
                    regs = [(r[0], int(r[1]), int(r[2])) for r in _REGS.findall(args)]
                    if st and len(regs) == 4:
                        f, bank, lo, hi, _ = st
                        b, l, h = regs[3]
                        if f != _format(op) and b == bank and l <= hi and lo <= h:
                            bad.add((name, off, op))
                    st = (_format(op),) + regs[0] + (0,)
                elif st:
                    w = st[4] + (int(args.split()[0], 0) + 1 if op == "s_nop" else 1)
                    st = st[:4] + (w,) if w < WAIT else None
                if target is not None and target in at:
                    work.append((at[target], st))
                if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                    break
                i += 1
        found += sorted(bad)
    return found


def check(obj: str):
    """Raise if a kernel in the object file holds an unguarded pair."""
    bad = adjacent_formats(disassemble(obj))
    if bad:
        raise RuntimeError("%s: matrix products of two formats follow each other on one accumulator:\n%s"
                           % (obj, "\n".join("  %s + %#x: %s" % b for b in bad)))
