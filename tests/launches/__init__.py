"""Launches of a library call, looked at without a GPU.

`record(code)` runs Python code in a process of its own, in which the HIP
runtime's entry points are those of hip_stub.c: every launch is recorded and
nothing runs, so the pointers that a call is given need not be memory.  The code
finds `fhtp` (the binding) and `PTR`, a fake aligned device pointer; its launches
come back as (kernel, grid, block), the kernel by its name and template arguments.
"""

import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))

_PROGRAM = """
import ctypes, json, sys
stub = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
stub.stub_name.restype = ctypes.c_char_p
from paper_1912_01884_amd import fhtp
PTR = 1 << 40
fhtp.lib()
def take():
    out = [(stub.stub_name(q).decode(), stub.stub_grid(q) & 0xffffffff, stub.stub_block(q))
           for q in range(stub.stub_launches())]
    stub.stub_reset()
    return out
def batch(shapes, bends):
    '''detect_batch of images (h, w, k, dtype) under bends (a fhtp.Bend each).'''
    jobs = [fhtp.Job(PTR, d, h, w, k, b, PTR, PTR) for (h, w, k, d), b in zip(shapes, bends)]
    arr = (fhtp.Job * len(jobs))(*jobs)
    n = fhtp.batch_workspace_bytes(jobs)
    fhtp._check(fhtp.lib().fhtp_detect_batch(arr, len(jobs), PTR, n, None), "detect_batch")
    return take()
def detect(h, w, k, dtype, bend, opt=None):
    n = fhtp.detect_ex_workspace_bytes(dtype, h, w, k, bend, opt)
    fhtp._check(fhtp.lib().fhtp_detect_polyline_ex(
        PTR, dtype, h, w, k, bend, None if opt is None else ctypes.byref(opt), PTR, n, PTR, PTR,
        None), "detect_polyline_ex")
    return take()
results = []
"""


def record(code, tmp_path):
    """The list `results` that `code` filled."""
    stub = os.path.join(str(tmp_path), "libhip_stub.so")
    if not os.path.exists(stub):
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-Wall", os.path.join(HERE, "hip_stub.c"),
                        "-o", stub], check=True)
    prog = _PROGRAM + code + "\nprint(json.dumps(results))\n"
    r = subprocess.run([sys.executable, "-c", prog, stub], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout.strip().splitlines()[-1])


def name(mangled):
    """`kernel` of a recorded kernel name (_ZN...kernelI<template arguments>E...)."""
    out = subprocess.run(["c++filt", mangled], capture_output=True, text=True).stdout.strip()
    return out.split("(anonymous namespace)::", 1)[-1].split("<", 1)[0].split("(", 1)[0]
