"""The HIP calls that the library's host code makes, written down on the CPU (tests/hip_calls/recorder.c).

``run(program)`` runs Python source in a process of its own with the recorder in front of the HIP runtime;
there ``L`` is the library, ``P`` an address that nothing looks at, ``params(...)`` a pointer to
``nvfp4_46_params``, and ``calls()`` the calls since it was last asked: (kind, kernel, bytes, grid, stream).
What the program assigns to ``result`` (JSON's types) is returned.
"""
from __future__ import annotations

import json
import os
import subprocess
import sys
from pathlib import Path

_HERE = Path(__file__).resolve().parent / "hip_calls"
_SO = _HERE / "_build" / "librecorder.so"
_ROOT = _HERE.parent.parent

_PROLOGUE = """
import ctypes as C, json
from paper_2512_02010_amd import binding as B
class Call(C.Structure):
    _fields_ = [("kind", C.c_int32), ("grid", C.c_int32), ("kernel", C.c_void_p), ("bytes", C.c_int64), ("stream", C.c_void_p)]
KINDS = {1: "set_attribute", 2: "launch", 3: "get_device", 4: "device_attribute", 5: "symbol_address"}
recorder, room = C.CDLL(None), (Call * 4096)()
def calls():
    n = recorder.recorded(room)
    return [(KINDS[c.kind], c.kernel or 0, c.bytes, c.grid, c.stream or 0) for c in room[:n]]
L, P = B.lib(), 1 << 20
def params(rows, cols, **kw):
    return C.byref(B.make_params(rows, cols, **kw))
calls()
"""


def _build() -> Path:
    source = _HERE / "recorder.c"
    if not _SO.exists() or _SO.stat().st_mtime < source.stat().st_mtime:
        _SO.parent.mkdir(parents=True, exist_ok=True)
        tmp = _SO.with_suffix(f".tmp{os.getpid()}.so")
        subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-fPIC", "-shared", str(source), "-o", str(tmp)], check=True)
        os.replace(tmp, _SO)
    return _SO


def run(program: str):
    env = dict(os.environ, LD_PRELOAD=str(_build()))
    r = subprocess.run([sys.executable, "-c", _PROLOGUE + program + "\nprint('RESULT' + json.dumps(result))"], cwd=_ROOT, env=env,
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.rsplit("RESULT", 1)[1])
