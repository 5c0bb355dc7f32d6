"""What the expert kernel takes for granted of the compiler, checked in the AMD code objects of the library just built.

Placement: the kernel's two LDS buffers for token rows are the destination of direct-to-LDS loads, whose LDS address is 16
bits wide, so they have to lie in the first 64 KiB.  The language does not say where a __shared__ array goes.  Both are
aligned to kStageAlign and the kernel's other arrays are smaller than that together: whatever lies ahead of or between
the buffers moves the end of the segment by a whole kStageAlign, and the segment's size shows it.
"""
from __future__ import annotations

import os
import re
import subprocess
import tempfile

LLVM = os.environ.get("ROCM_LLVM_BIN", "/opt/rocm/llvm/bin")
KERNEL = "ffn_kernel"
STAGE_END = 65536     # 2 * kStageBuffer
STAGE_ALIGN = 4096    # kStageAlign


def _run(tool, *args, cwd=None):
    return subprocess.run([os.path.join(LLVM, tool), *args], cwd=cwd, capture_output=True, text=True, check=True).stdout


def code_object_texts(lib_path: str):
    """The metadata notes of every gfx950 code object in the library that holds the kernel."""
    with tempfile.TemporaryDirectory() as d:
        os.symlink(os.path.abspath(lib_path), os.path.join(d, "lib.so"))   # (the extracted objects land beside it)
        _run("llvm-objdump", "--offloading", "lib.so", cwd=d)
        for name in sorted(os.listdir(d)):
            if not name.endswith("gfx950"):
                continue
            notes = _run("llvm-readelf", "--notes", name, cwd=d)
            if KERNEL in notes:
                yield notes


def check_placement(notes: str) -> int:
    """Raises if an LDS buffer of the kernel can reach past STAGE_END; the number of kernels looked at."""
    kernels = re.findall(r"\.group_segment_fixed_size:\s*(\d+)(?:(?!\.group_segment_fixed_size).)*?\.name:\s*(\S*" + KERNEL + r"\S*)",
                         notes, re.S)
    for size, name in kernels:
        if not STAGE_END <= int(size) < STAGE_END + STAGE_ALIGN:
            raise RuntimeError(f"{name}: {size} bytes of LDS: the buffers for token rows do not lie in the first {STAGE_END}")
    return len(kernels)


def check(lib_path: str) -> None:
    n = 0
    for notes in code_object_texts(lib_path):
        n += check_placement(notes)
    if n == 0:
        raise RuntimeError(f"{lib_path}: no {KERNEL} found")
