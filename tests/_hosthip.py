"""The library's host side on the CPU, over the recording runtime of
_host_hip.cpp (not collected).  run(code) executes `code` in a process of its
own, where `cc` is the binding, `ctx` a context on the recorded device,
log() / clear() / fail(name) read and reset the record or make an allocation
fail and copied() is what the last synchronous copy moved (a plan's programs);
what `code` leaves in `result` comes back."""
import json
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_SRC = os.path.join(ROOT, "tests", "_host_hip.cpp")
_DIR = None

_PRELUDE = """
import ctypes, json, sys
sys.path.insert(0, {root!r})
_rt = ctypes.CDLL({stub!r}, mode=ctypes.RTLD_GLOBAL)
_rt.host_hip_log.restype = ctypes.c_char_p
import numpy as np
import paper_2303_10788_amd as cc

class _Ctx:
    pass

def new_context(**fields):
    o = cc.ccut_opts()
    for k, v in fields.items():
        setattr(o, k, v)
    c = _Ctx()
    c.handle = cc.ccut_ctx_create(o)
    return c

log = lambda: [l.split() for l in _rt.host_hip_log().decode().splitlines()]
clear = _rt.host_hip_clear
fail = lambda name: _rt.host_hip_fail(name.encode())

def copied():
    n = ctypes.c_size_t()
    _rt.host_hip_copied.restype = ctypes.c_void_p
    p = _rt.host_hip_copied(ctypes.byref(n))
    return ctypes.string_at(p, n.value)

ctx = new_context()
result = None
"""


def run(code):
    global _DIR
    if _DIR is None:
        from paper_2303_10788_amd import build as B
        _DIR = tempfile.TemporaryDirectory()
        subprocess.run([B.hipcc(), "-no-hip-rt", "-x", "c++", "-O1", "-std=c++17", "-fPIC", "-shared",
                        "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", _SRC, "-o",
                        os.path.join(_DIR.name, "host_hip.so")], check=True, capture_output=True)
    full = _PRELUDE.format(root=ROOT, stub=os.path.join(_DIR.name, "host_hip.so")) + code
    full += "\nsys.stdout.write('\\n' + json.dumps(result))\nsys.stdout.flush()\nimport os\nos._exit(0)\n"
    r = subprocess.run([sys.executable, "-c", full], capture_output=True, text=True, timeout=240)
    assert r.returncode == 0, r.stderr[-3000:]
    return json.loads(r.stdout.strip().splitlines()[-1])


def launches_before(log):
    """Per launch (stream, kernel, grid, block, the set of launches that are
    sure to have ended when it starts): stream order, events and the waits of
    the host."""
    done, events, host, out = {}, {}, set(), []
    for e in log:
        s = e[1] if len(e) > 1 else None
        if e[0] == "launch":
            before = done.get(s, set()) | host
            out.append((s, e[2], int(e[3]), int(e[4]), before))
            done[s] = before | {len(out) - 1}
        elif e[0] == "record":
            events[e[2]] = set(done.get(s, set())) | host
        elif e[0] == "wait":
            done[s] = done.get(s, set()) | events.get(e[2], set())
        elif e[0] == "sync":
            host = host | done.get(s, set())
        elif e[0] == "waited":
            host = host | events.get(s, set())
    return out
