"""What the expert kernel takes for granted of the compiler, checked in the AMD code objects of the library just built.

Placement: the kernel's two LDS buffers for token rows are the destination of direct-to-LDS loads, whose LDS address is 16
bits wide, so they have to lie in the first 64 KiB.  The language does not say where a __shared__ array goes.  Both are
aligned to kStageAlign and the kernel's other arrays are smaller than that together: whatever lies ahead of or between
the buffers moves the end of the segment by a whole kStageAlign, and the segment's size shows it.

Waits: a wave reports its pieces of a chunk of token rows at a barrier, before which they must have landed.  The kernel waits
until at most as many loads are outstanding as it has issued behind them, a number that follows from its source as long as
the compiler neither drops nor merges loads.  They are counted again in the machine code, ahead of every barrier behind a
direct-to-LDS load, in the order of the listing (the kernel's loops around them are laid out straight).

Products: the wide kernel's matrix instructions are written out, so the compiler does not keep the wait states that they need: two
between a VALU instruction that writes an operand of theirs and its use, and up to 19 (for the longest of them) between a product and
any other instruction on its sums.  Their operands come from loads and their sums stay in place; that no instruction comes too
close is checked in the machine code, in the order of the listing and across every branch.
"""
from __future__ import annotations

import os
import re
import subprocess
import tempfile

LLVM = os.environ.get("ROCM_LLVM_BIN", "/opt/rocm/llvm/bin")
KERNEL = "ffn_kernel"
WIDE = "ffn_wide_kernel"
STAGE_END = 65536     # 2 * kStageBuffer
STAGE_ALIGN = 4096    # kStageAlign


def _run(tool, *args, cwd=None):
    return subprocess.run([os.path.join(LLVM, tool), *args], cwd=cwd, capture_output=True, text=True, check=True).stdout


def code_object_texts(lib_path: str):
    """(metadata notes, disassembly) of every gfx950 code object in the library that holds the kernel."""
    with tempfile.TemporaryDirectory() as d:
        os.symlink(os.path.abspath(lib_path), os.path.join(d, "lib.so"))   # (the extracted objects land beside it)
        _run("llvm-objdump", "--offloading", "lib.so", cwd=d)
        for name in sorted(os.listdir(d)):
            if not name.endswith("gfx950"):
                continue
            notes = _run("llvm-readelf", "--notes", name, cwd=d)
            if KERNEL in notes:
                yield notes, _run("llvm-objdump", "-d", name, cwd=d)


def check_placement(notes: str) -> int:
    """Raises if an LDS buffer of the kernel can reach past STAGE_END; the number of kernels looked at."""
    kernels = re.findall(r"\.group_segment_fixed_size:\s*(\d+)(?:(?!\.group_segment_fixed_size).)*?\.name:\s*(\S*" + KERNEL + r"\S*)",
                         notes, re.S)
    for size, name in kernels:
        if not STAGE_END <= int(size) < STAGE_END + STAGE_ALIGN:
            raise RuntimeError(f"{name}: {size} bytes of LDS: the buffers for token rows do not lie in the first {STAGE_END}")
    return len(kernels)


def check_waits(listing: str) -> int:
    """Raises if a barrier of the kernel can be reached before the direct-to-LDS loads ahead of it have landed; the number of
    such barriers."""
    barriers = 0
    name = ""
    behind = None         # memory operations issued behind the last direct-to-LDS load, None = none to wait for
    landed = False
    for line in listing.splitlines():
        head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if head:
            name, behind = head.group(1), None
            continue
        words = line.split("//")[0].split()
        if not words or KERNEL not in name:
            continue
        op = words[0]
        if op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            if words[-1] == "lds":
                behind, landed = 0, False
            elif behind is not None:
                behind += 1
        elif op == "s_waitcnt" and behind is not None:
            count = re.search(r"vmcnt\((\d+)\)", line)
            landed = landed or (count is not None and int(count.group(1)) <= behind)
        elif op == "s_barrier" and behind is not None:
            if not landed:
                raise RuntimeError(f"{name}: a barrier {behind} loads behind direct-to-LDS loads that nothing waits for")
            barriers += 1
            behind = None
    return barriers


SUM_STATES = 19       # most wait states between a product and another instruction on its sums
OPERAND_STATES = 2    # between a VALU instruction and a product that takes what it writes


def _registers(operand: str) -> set:
    m = re.fullmatch(r"-?\|?([va])(?:\[(\d+):(\d+)\]|(\d+))\|?", operand)
    if not m:
        return set()
    lo = int(m.group(2) or m.group(4))
    return {(m.group(1), i) for i in range(lo, int(m.group(3) or lo) + 1)}


class _Instruction:
    """What the products' wait states depend on, from a line of the listing."""

    def __init__(self, line: str):
        words = line.split("//")[0].replace(",", " ").split()
        self.text, op = line.strip(), words[0]
        self.product = op.startswith("v_mfma")
        self.states = int(words[1], 0) + 1 if op == "s_nop" else 1
        self.regs = set().union(*map(_registers, words[1:]))
        self.sums = _registers(words[1]) if self.product else set()
        self.writes = set()
        if op.startswith("v_") and not self.product and not op.startswith("v_cmp"):
            self.writes = _registers(words[1])
            if "swap" in op:      # (writes both operands)
                self.writes |= _registers(words[2])
        self.ends = op in ("s_branch", "s_endpgm", "s_setpc_b64")
        m = re.search(r"//\s*([0-9A-Fa-f]+):", line)
        self.address = int(m.group(1), 16) if m else None
        m = re.search(r"<\S+?(?:\+0x([0-9a-f]+))?>\s*$", line) if op.startswith(("s_branch", "s_cbranch")) else None
        self.jump = int(m.group(1) or "0", 16) if m else None     # from the start of the function


def _check_distances(ins: _Instruction, recent: list):
    states = 0
    for before in reversed(recent):
        if states >= SUM_STATES:
            return
        if ins.product and states < OPERAND_STATES and before.writes & ins.regs:
            raise RuntimeError(f"{ins.text} uses a register that was written {states} states before")
        if not ins.product and before.sums & ins.regs:
            raise RuntimeError(f"{ins.text} uses a sum of a product {states} states before")
        states += before.states


def _check_function(name: str, start: int, code: list):
    at = {ins.address: i for i, ins in enumerate(code) if ins.address is not None}
    paths = [(0, [], None)]       # where a path begins, what ran before it, how many states it is followed for (None: to the end)
    while paths:
        i, recent, left = paths.pop()
        while i < len(code) and (left is None or left > 0):
            ins = code[i]
            try:
                _check_distances(ins, recent)
            except RuntimeError as e:
                raise RuntimeError(f"{name}: {e}") from None
            recent = recent[-SUM_STATES:] + [ins]
            if left is not None:
                left -= ins.states
            if ins.jump is not None:
                if start + ins.jump not in at:
                    raise RuntimeError(f"{name}: {ins.text}: no instruction at its target")
                if left is None or left > 0:
                    paths.append((at[start + ins.jump], recent, SUM_STATES if left is None else left))
            if ins.ends:
                if left is not None:
                    break
                recent = []
            i += 1


def check_operands(listing: str) -> int:
    """Raises if an instruction of the wide kernel comes too close to a matrix instruction (see above); the number of matrix
    instructions."""
    products = 0
    name, start, code = "", 0, []

    def finish():
        nonlocal products
        if WIDE in name:
            _check_function(name, start, code)
            products += sum(ins.product for ins in code)

    for line in listing.splitlines():
        head = re.match(r"([0-9a-f]+) <(\S+)>:", line)
        if head:
            finish()
            name, start, code = head.group(2), int(head.group(1), 16), []
        elif WIDE in name and line.split("//")[0].strip():
            code.append(_Instruction(line))
    finish()
    return products


def check(lib_path: str) -> None:
    kernels = barriers = products = 0
    for notes, listing in code_object_texts(lib_path):
        kernels += check_placement(notes)
        barriers += check_waits(listing)
        products += check_operands(listing)
    if kernels == 0 or barriers < kernels or products == 0:
        raise RuntimeError(f"{lib_path}: {kernels} kernels, {barriers} barriers and {products} products found: the checks do not read this library")
