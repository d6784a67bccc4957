"""Builds ffn_host.cpp: the device code of the FFN kernels on the host, its
LDS accesses handed to a recorder.  Used by the CPU tests of the FFN launch."""

import ctypes
import os
import re
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2505_08944_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


def _device_part():
    """k_ffn.hip up to its host launchers, LDS accesses as recorder calls."""
    src = open(os.path.join(CSRC, "k_ffn.hip")).read()
    head, rest = src.split("hipError_t launch_ffn(", 1)
    assert "<<<" not in head and "<<<" in rest

    def sub(pattern, repl, text, n, flags=0):
        out, k = re.subn(pattern, repl, text, flags=flags)
        assert k == n if n else k > 0, (pattern, k)
        return out

    # the direct load (its last operand is the LDS address), then the empty fences
    head = sub(r'asm volatile\("s_mov_b32 m0.*?\);', "lds_load(lds_addr);", head, 1, re.S)
    head = sub(r'asm volatile\("".*?\);', ";", head, 0)
    head = sub(r"\*reinterpret_cast<const (bf16x8_t|uint4)\*>\(q", r"lds_read<\1>(q", head, 3)
    head = sub(r"volatile __attribute__\(\(address_space\(3\)\)\) int\* flag =.*?;", "const LdsFlag flag(smem);",
               head, 1, re.S)
    assert "asm" not in re.sub(r"//.*", "", head)
    return head + "\n}  // namespace aep\n"


def load():
    if not os.path.exists(CLANG):
        pytest.skip("needs ROCm's clang++ as the host compiler")
    with tempfile.TemporaryDirectory() as tmp:
        os.mkdir(os.path.join(tmp, "hip"))
        open(os.path.join(tmp, "hip", "hip_runtime.h"), "w").close()  # the mock stands in ffn_host.cpp
        with open(os.path.join(tmp, "ffn_device.inc"), "w") as f:
            f.write(_device_part())
        so = os.path.join(tmp, "ffn_host.so")
        subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-I", tmp, "-I", CSRC,
                        os.path.join(HERE, "ffn_host.cpp"), "-o", so], check=True)
        return ctypes.CDLL(so)
