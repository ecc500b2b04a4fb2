"""The library on a recording stand-in for the HIP runtime (tests/hip_recorder.c):
host code alone, no GPU.  Runs a piece of Python in a process of its own, with

  rec      the stand-in (clear(), launches() -> [(kernel, workgroups, threads)], fail(name, times))
  mls      the binding, loaded on it, and L its C entry points
  step_buffers(n)   an mls_step_buffers whose arrays are never read

and returns what it assigns to `result`.
"""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

_HEAD = r"""
import ctypes, json, re, sys
sys.path.insert(0, %r)
_r = ctypes.CDLL(%r, mode=ctypes.RTLD_GLOBAL)
_r.rec_name.restype = ctypes.c_char_p
import numpy as np
from paper_1805_01113_amd import mls, workloads as W
L = mls.load(need_torch=False)


class rec:
    clear = staticmethod(_r.rec_clear)

    @staticmethod
    def launches():
        out = []
        for i in range(_r.rec_count()):
            m = re.search(r"\d+(k_[a-z0-9_]+?)(?:E|IL)", _r.rec_name(i).decode())
            out.append((m.group(1), _r.rec_grid(i), _r.rec_threads(i)))
        return out

    @staticmethod
    def fail(name, times=1):
        _r.rec_fail(name.encode(), times)


_any = ctypes.create_string_buffer(1 << 12)
ptr = ctypes.addressof(_any)


def step_buffers(n):
    b = mls._StepBuf()
    b.n = n
    for k, _ in mls._StepBuf._fields_[1:]:
        setattr(b, k, ptr)
    return b


result = None
"""


def build(folder):
    so = os.path.join(str(folder), "hip_recorder.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "hip_recorder.c"), "-o", so])
    return so


def run(folder, code):
    so = build(folder)
    p = subprocess.run([sys.executable, "-c", _HEAD % (ROOT, so) + code + "\nprint('RESULT ' + json.dumps(result))"],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    lines = [s for s in p.stdout.splitlines() if s.startswith("RESULT ")]
    assert p.returncode == 0 and lines, p.stdout[-3000:]
    return json.loads(lines[-1][7:])
