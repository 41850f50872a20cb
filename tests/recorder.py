"""What the library's calls enqueue, looked at without a GPU.

`run(script)` runs Python statements in a process of its own whose HIP runtime is
the recorder of hip_recorder.c: kernels, event records and stream waits are noted
and nothing runs.  The statements see P (the binding, with numbers in the place
of device tensors), C (the workloads), `lib` (the C ABI), `calls(fn)` (the
records of fn()) and `fail_at(n)`, and give `out` back.
"""
import json
import os
import subprocess
import sys
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2002_07401_amd", "libqmc_jagp.so")

_PRELUDE = """
import ctypes, json, re, sys, types
sys.path.insert(0, {root!r}); sys.path.insert(0, {here!r})
rec = ctypes.CDLL({stub!r}, mode=ctypes.RTLD_GLOBAL)
rec.rec_get.restype = ctypes.c_char_p
torch = types.ModuleType("torch")   # (its libraries would bring the real runtime along)
torch.Tensor = object
torch.float64 = "float64"
torch.autograd = types.SimpleNamespace(Function=object)
torch.cuda = types.SimpleNamespace(Stream=object)
sys.modules["torch"] = torch
import numpy as np
from workloads import configs as C
import paper_2002_07401_amd as P
lib = P.load()
vp = ctypes.c_void_p
def dev(n):   # an address that no call reads
    return vp(0x10000000 + 256 * n)
def records():
    return [rec.rec_get(i).decode() for i in range(rec.rec_count())]
def calls(fn):
    rec.rec_clear()
    fn()
    return records()
def kernels(fn):   # (name, grid, block) of each launch
    o = []
    for r in calls(fn):
        f = r.split()
        if f[0] == "launch":
            name = re.sub(r"^_ZN3qmcL?\\d+", "", f[1])
            o.append((name, tuple(map(int, f[2].split(","))), tuple(map(int, f[3].split(",")))))
    return o
def fail_at(n):
    rec.rec_fail_at(ctypes.c_long(n))
def ok(code):
    assert code == 0, lib.qmc_last_error()
out = None
"""


def run(script, timeout=120):
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    with tempfile.TemporaryDirectory() as td:
        stub = os.path.join(td, "libhiprec.so")
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", stub, os.path.join(HERE, "hip_recorder.c")], check=True)
        code = _PRELUDE.format(root=ROOT, here=HERE, stub=stub) + script + "\nprint('@@' + json.dumps(out))\n"
        res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=timeout)
        assert res.returncode == 0, res.stderr[-4000:]
        return json.loads(res.stdout.split("@@")[-1])
