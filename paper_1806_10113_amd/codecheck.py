"""Check of built device code for one form that MI355X executes wrongly.

A 64-bit vector shift (v_lshlrev_b64, v_lshrrev_b64, v_ashrrev_i64) whose amount
lies in the last vector register that its wave has takes a wrong amount as soon as
waves share a SIMD (here: 15 % of 419 M such shifts with 4,096 blocks resident in
turn, none with 64 blocks, none with the amount one register lower; products,
conversions and additions with a 32-bit source there are right).  Waves get their
registers in units of eight, so it takes a kernel whose register count is a multiple
of eight and a compiler that puts an amount into the last one; hipcc does not avoid
it for gfx950.  Totals of the memory-limited walk were off by it when its registers
were capped at 80.  The build fails on such code: another cap (waves per SIMD),
depth or scheduler for the kernel named lets the registers fall elsewhere.
"""
from __future__ import annotations

import os
import re
import struct
import subprocess
import tempfile

ARCH = "gfx950"
LLVM = os.environ.get("ROCM_LLVM_BIN", "/opt/rocm/llvm/bin")
_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
_SHIFT = re.compile(r"\s(v_(?:lshlrev_b64|lshrrev_b64|ashrrev_i64)\S*\s+v\[\d+:\d+\],\s*v(\d+),.*?)\s*(?://.*)?$")


def code_objects(path: str) -> list:
    """The gfx950 code objects in a host object or library (bytes each)."""
    blob = open(path, "rb").read()
    out, at = [], blob.find(_MAGIC)
    while at >= 0:
        pos = at + len(_MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", blob, pos - 8)[0]):
            off, size, length = struct.unpack_from("<QQQ", blob, pos)
            if ARCH.encode() in blob[pos + 24:pos + 24 + length]:
                out.append(blob[at + off:at + off + size])
            pos += 24 + length
        at = blob.find(_MAGIC, pos)
    return out


def last_registers(notes: str) -> dict:
    """Kernel -> index of the last vector register of its allocation."""
    found = re.findall(r"\.symbol:\s*'?(\S+?)\.kd'?\s.*?\.vgpr_count:\s*(\d+)", notes, re.S)
    return {name: (max(int(count), 1) + 7) // 8 * 8 - 1 for name, count in found}


def bad_shifts(listing: str, last: dict) -> list:
    """(kernel, instruction) of every shift whose amount is in that register."""
    out, kernel = [], None
    for line in listing.splitlines():
        head = re.match(r"[0-9a-f]+ <(\S+)>:$", line)
        if head:
            kernel = head.group(1)
            continue
        shift = _SHIFT.search(line)
        # (code outside the kernels would run with its caller's registers: none here)
        if shift and int(shift.group(2)) == last.get(kernel, -1):
            out.append((kernel, shift.group(1)))
    return out


def scan(path: str) -> tuple:
    """(kernels seen, bad shifts) of a host object or library."""
    kernels, bad = 0, []
    for code in code_objects(path):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(code)
            f.flush()
            run = lambda *a: subprocess.run(a, capture_output=True, text=True, check=True).stdout
            last = last_registers(run(os.path.join(LLVM, "llvm-readelf"), "--notes", f.name))
            kernels += len(last)
            bad += bad_shifts(run(os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", f.name), last)
    return kernels, bad
