"""What the library launches for given sizes, on the CPU: the calls run in a process that has launch_recorder.c loaded in the
place of the HIP runtime, so every host-side rule runs and no kernel does."""
from __future__ import annotations

import json
import os
import re
import subprocess
import sys
import tempfile
from collections import namedtuple

from paper_2211_10017_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
Launch = namedtuple("Launch", "kernel grid block shared device")     # kernel: demangled, with its template arguments
Call = namedtuple("Call", "rc launches raised noted")                # raised: (kernel, device) of each LDS limit asked for
P = "ptr"                                                            # a buffer that nothing reads
_SIZE = 1 << 40                                                      # workspaces: as large as anything asks for

_CHILD = r"""
import ctypes, json, sys
shim, lib_path = sys.argv[1:3]
rec = ctypes.CDLL(shim, mode=ctypes.RTLD_GLOBAL)
rec.recorder_take.restype = ctypes.c_char_p
lib = ctypes.CDLL(lib_path)
lib.moe_last_ffn_kernels.restype = ctypes.c_char_p
conv = lambda a: ctypes.c_void_p(0x10000) if a == "ptr" else ctypes.c_void_p(None) if a is None else ctypes.c_size_t(a[0]) if isinstance(a, list) else ctypes.c_size_t(a) if a >= 1 << 31 else ctypes.c_int(a)
out = []
for name, device, args in json.load(sys.stdin):
    rec.recorder_device(device)
    rec.recorder_clear()
    rc = getattr(lib, name)(*[conv(a) for a in args])
    out.append([rc, rec.recorder_take().decode(), lib.moe_last_ffn_kernels().decode()])
json.dump(out, sys.stdout)
"""
_shim = None


def _build():
    global _shim
    if _shim is None:
        _shim = tempfile.TemporaryDirectory(prefix="launch_recorder_")
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", os.path.join(_shim.name, "rec.so"), os.path.join(HERE, "launch_recorder.c")], check=True)
    return os.path.join(_shim.name, "rec.so")


def record(calls, lib=B.LIB_PATH):
    """calls: (entry point, arguments[, device]) each; returns a Call for each."""
    calls = [(c[0], c[2] if len(c) > 2 else 0, list(c[1])) for c in calls]
    r = subprocess.run([sys.executable, "-c", _CHILD, _build(), lib], input=json.dumps(calls), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    rows = json.loads(r.stdout)
    names = sorted({line.split()[-1] for _, text, _ in rows for line in text.splitlines()})
    plain = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True, check=True).stdout.splitlines()
    # "void moe::kernel<4, (moe::Mode)1>(moe::Args)" -> "kernel<4, 1>"
    shown = {m: re.sub(r"\(moe::\w+\)(?=\d)", "", p).replace("void ", "").replace("moe::", "").split("(")[0] for m, p in zip(names, plain)}
    out = []
    for rc, text, noted in rows:
        launches, raised = [], []
        for f in (line.split() for line in text.splitlines()):
            if f[0] == "launch":
                launches.append(Launch(shown[f[7]], tuple(map(int, f[2:5])), int(f[5]), int(f[6]), int(f[1])))
            else:
                raised.append((shown[f[3]], int(f[1])))
        out.append(Call(rc, launches, raised, noted))
    return out


def gate(T, d, E, act=B.MOE_F16, k=2):
    return "moe_gate_topk", [P, act, P, None, None, T, d, E, k, 1, P, P, None]


def permute(T, k, E, d=0):
    return "moe_permute", [P, P if d else None, B.MOE_F16, T, k, E, d or 64, P if d else None, P, P, P, P, _SIZE, None]


def ffn(R, E, d, F, bits, g=0, act=B.MOE_F16, bound=0, activation=0, y=B.MOE_F32):
    return "moe_grouped_ffn_wq", [P, act, P, R, E, bound, d, F, bits, g, activation, P, P, None, P, P, None, P, y, P, _SIZE, None]


def indexed(R, E, k, d, F, bits, g=0, act=B.MOE_F16, bound=0, scale=False):
    return "moe_grouped_ffn_wq_indexed", [P, act, P, k, P if scale else None, P, R, E, bound, d, F, bits, g, 0, P, P, None, P, P, None, P, B.MOE_F32, P, _SIZE, None]


def unsorted(T, k, E, d, F, bits, g=0, act=B.MOE_F16, scale=False, idx=P):
    return "moe_grouped_ffn_wq_unsorted", [P, act, idx, P if scale else None, T, k, E, d, F, bits, g, 0, P, P, None, P, P, None, P, B.MOE_F32, P, P, P, P, _SIZE, None]


def sliced(T, k, E, d, F, bits, g=0, act=B.MOE_F16, out=B.MOE_F32):
    return "moe_grouped_ffn_wq_sliced", [P, act, P, P, T, k, E, d, F, bits, g, 0, P, P, None, P, P, None, P, out, P, P, P, P, _SIZE, None]


def gated(T, k, E, d, F, bits, scale=True, workspace=_SIZE):
    return "moe_grouped_ffn_wq_gated", [P, B.MOE_F16, P, P if scale else None, T, k, E, d, F, bits, 0, 0, P, P, None, P, P, None, P, B.MOE_F32, P, P, P, P, [workspace], None]
