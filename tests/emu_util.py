"""Kernel sources built for the CPU (tests/emu/hip/hip_runtime.h): what depends on
the order in which the waves of a workgroup run shows here every time."""
from __future__ import annotations

import ctypes
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_06467_amd", "csrc")
CLANG = os.environ.get("EMU_CXX", "/opt/rocm/bin/amdclang++")

# bf16 rounding for hosts whose runtime library lacks it (round to nearest even)
_PRELUDE = """
extern "C" __bf16 __truncsfbf2(float f) {
    unsigned u = __builtin_bit_cast(unsigned, f);
    u = (u & 0x7fffffffu) > 0x7f800000u ? u | 0x400000u : u + 0x7fffu + ((u >> 16) & 1u);
    return __builtin_bit_cast(__bf16, (unsigned short)(u >> 16));
}
"""


def build(tmp, source: str, wrappers: str) -> ctypes.CDLL:
    """csrc/<source> with its launches turned into loops, and C wrappers, as a library."""
    if not os.path.exists(CLANG):
        pytest.skip("needs a clang that knows bf16 vectors")
    with open(os.path.join(CSRC, source)) as f:
        text = f.read()
    text = re.sub(r"(\w+(?:<[^<>\n]*>)?)<<<(.*?)>>>\((\w+)\)",
                  r"emu::launch([&] { (\1)(\3); }, \2)", text, flags=re.S)
    cpp, so = os.path.join(tmp, "emu.cpp"), os.path.join(tmp, "emu.so")
    with open(cpp, "w") as f:
        f.write(_PRELUDE + text + wrappers)
    r = subprocess.run([CLANG, "-std=c++17", "-O1", "-w", "-fPIC", "-shared", "-I",
                        os.path.join(ROOT, "tests", "emu"), "-I", CSRC, cpp, "-o", so],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return ctypes.CDLL(so)
