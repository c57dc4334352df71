"""What a call of the library launches, seen on the CPU.

`recorder/recorder.cpp` is a stand-in for the HIP runtime that records kernel
launches and runs none.  `start(tmp)` builds it; `run(recorder, source)` runs
Python source in a process of its own in which the library is bound to the
recorder: `B` is the binding, `call(...)` makes one call with made-up device
addresses and `launches()` returns what has been launched since it was last
asked, as (kernel, grid, block, thread).  The source's `result` comes back.
"""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_PRELUDE = r'''
import ctypes, json, os, re, sys, types
recorder = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
torch = types.ModuleType("torch")   # the binding imports it to load its HIP runtime first
torch._C = None
sys.modules["torch"] = torch
from paper_2609_07536_amd import binding as B
L = B.lib()
recorder.recorder_fail.argtypes = [ctypes.c_char_p]

def launches():
    n, out = recorder.recorder_count(), []
    name = ctypes.create_string_buffer(4096)
    grid, block, thread = ctypes.c_uint(), ctypes.c_uint(), ctypes.c_size_t()
    for i in range(n):
        recorder.recorder_get(i, name, 4096, ctypes.byref(grid), ctypes.byref(block),
                              ctypes.byref(thread))
        k = name.value.decode().replace("(anonymous namespace)::", "").replace("void ", "")
        out.append((re.sub(r"\(.*", "", k), grid.value, block.value, thread.value))
    recorder.recorder_clear()
    return out

ADDR = 1 << 32   # device addresses of launches that never run
def call(op, T, H, I, E, topk, splits=1, rows=0, C=0, mode=0, ws=ADDR, trace=False, counts=None):
    """One call; its return value."""
    wl, keep = B.make_workload(T, H, I, E, topk, splits, counts, rows=rows)
    w = ctypes.byref(wl)
    if op == "gemm1":
        return L.moe_gemm1_swiglu(ADDR, ADDR, ADDR, ADDR, ADDR, w, ws, 512, None)
    if op == "layer":
        return L.moe_layer_forward(ADDR, ADDR, ADDR, ADDR, ADDR, ADDR, ADDR, w, C, ws, 1 << 50, None)
    if op == "noalloc":
        return L.moe_gemm2_combine_noalloc(ADDR, ADDR, ADDR, ADDR, ADDR, ADDR, w, C, mode, None)
    return L.moe_gemm2_combine_ex(ADDR, ADDR, ADDR, ADDR, ADDR, ADDR, w, C, mode, ws, 1 << 50,
                                  None, ADDR if trace else None, 1 << 50)
'''


def start(tmp):
    gxx = shutil.which("g++")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if gxx is None or not os.path.isdir(os.path.join(rocm, "include", "hip")):
        pytest.skip("g++ or the HIP headers not available")
    src = os.path.join(ROOT, "tests", "recorder")
    out = str(tmp / "librecorder.so")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                        "-I", os.path.join(rocm, "include"), os.path.join(src, "recorder.cpp"),
                        "-Wl,-soname,libamdhip64.so.7",
                        "-Wl,--version-script=" + os.path.join(src, "exports.map"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


def run(recorder, source, **env):
    clean = {k: v for k, v in os.environ.items() if not k.startswith("MOE_GEMM2_")}
    r = subprocess.run([sys.executable, "-c",
                        _PRELUDE + source + "\nprint(json.dumps(result))", recorder, ROOT],
                       capture_output=True, text=True, timeout=300, env={**clean, **env})
    assert r.returncode == 0, r.stderr[-4000:]
    return json.loads(r.stdout.strip().splitlines()[-1])
