"""What the expert kernel takes for granted of the compiler, checked in the AMD code objects of the library just built.

Placement: the kernel's two LDS buffers for token rows are the destination of direct-to-LDS loads, whose LDS address is 16
bits wide, so they have to lie in the first 64 KiB.  The language does not say where a __shared__ array goes.  Both are
aligned to kStageAlign and the kernel's other arrays are smaller than that together: whatever lies ahead of or between
the buffers moves the end of the segment by a whole kStageAlign, and the segment's size shows it.

Waits: a wave reports its pieces of a chunk of token rows at a barrier, before which they must have landed.  The kernel waits
until at most as many loads are outstanding as it has issued behind them, a number that follows from its source as long as
the compiler neither drops nor merges loads.  They are counted again in the machine code, ahead of every barrier behind a
direct-to-LDS load, in the order of the listing (the kernel's loops around them are laid out straight).

Operands: the wide kernel's matrix instructions are written out, so the compiler does not keep the two wait states between a VALU
instruction that writes an operand of theirs and its use.  Their operands come from loads; that no VALU instruction writes one
so late is checked in the machine code.
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


def _vector_registers(operand: str) -> set:
    m = re.fullmatch(r"v(?:\[(\d+):(\d+)\]|(\d+))", operand)
    if not m:
        return set()
    lo = int(m.group(1) or m.group(3))
    return set(range(lo, int(m.group(2) or lo) + 1))


def check_operands(listing: str) -> int:
    """Raises if a VALU instruction of the wide kernel writes an operand of a matrix instruction within two wait states of its
    use; the number of matrix instructions."""
    products = 0
    name = ""
    recent = []           # (wait states it stands for, vector registers that a VALU instruction writes)
    for line in listing.splitlines():
        head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
        if head:
            name, recent = head.group(1), []
            continue
        words = line.split("//")[0].replace(",", " ").split()
        if not words or WIDE not in name:
            continue
        op = words[0]
        if op.startswith("v_mfma"):
            products += 1
            states = 0
            for n, written in reversed(recent):
                if states >= 2:
                    break
                if written & (_vector_registers(words[2]) | _vector_registers(words[3])):
                    raise RuntimeError(f"{name}: {line.strip()} uses a register that was written {states} states before")
                states += n
        valu = op.startswith("v_") and not op.startswith(("v_mfma", "v_cmp", "v_readlane", "v_readfirstlane"))
        recent = recent[-3:] + [(int(words[1]) + 1 if op == "s_nop" else 1, _vector_registers(words[1]) if valu else set())]
    return products


def check(lib_path: str) -> None:
    kernels = barriers = products = 0
    for notes, listing in code_object_texts(lib_path):
        kernels += check_placement(notes)
        barriers += check_waits(listing)
        products += check_operands(listing)
    if kernels == 0 or barriers < kernels or products == 0:
        raise RuntimeError(f"{lib_path}: {kernels} kernels, {barriers} barriers and {products} products found: the checks do not read this library")
