"""Records the kernel launches of libbgpo calls on the CPU.

The calls run in a child process that has hip_recorder.c in its global symbol
scope, so the library's HIP calls reach the recorder and not the runtime: every
launch is held against the runtime's limits and noted, nothing runs, and no
pointer is followed.  Sizes that no memory holds can be checked that way.
"""
import ctypes
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2510_11683_amd", "libbgpo.so")


def build_recorder(path):
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-Werror", "-o", path,
                    os.path.join(HERE, "hip_recorder.c")], check=True)
    return path


def record(recorder, calls):
    """[(function, [argument, ..])] -> [{"status", "launches", "ms", "counts"}].

    Arguments: None, an int (int64), a float, "ptr" (a device address of its
    own, far from every other), ("prob", bytes), ("i32", int), "ws" (a workspace
    and its size, for the call's problem) or "timing" (a timing record)."""
    enc = [(f, [["prob", a[1].hex()] if isinstance(a, tuple) and a[0] == "prob" else a for a in args])
           for f, args in calls]
    r = subprocess.run([sys.executable, os.path.abspath(__file__), recorder, LIB], input=json.dumps(enc),
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout)


class _Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("grid", ctypes.c_uint32 * 3), ("block", ctypes.c_uint32 * 3)]


class _Timing(ctypes.Structure):
    _fields_ = [("ms", ctypes.c_double * 10), ("launches", ctypes.c_int64 * 10)]


def _child(recorder, lib_path):
    rec = ctypes.CDLL(recorder, mode=ctypes.RTLD_GLOBAL)
    lib = ctypes.CDLL(lib_path)
    launches = (_Launch * 65536).in_dll(rec, "rec_launches")
    count = ctypes.c_int.in_dll(rec, "rec_n_launches")
    out = []
    for fn, args in json.load(sys.stdin):
        rec.rec_reset()
        c, prob, timing = [], None, _Timing()
        for i, a in enumerate(args):
            if a == "ptr":
                c.append(ctypes.c_void_p((i + 1) << 44))
            elif a == "ws":
                n = ctypes.c_size_t(0)
                assert lib.bgpo_workspace_size(prob, ctypes.byref(n)) == 0, (fn, args)
                c += [ctypes.c_void_p((i + 1) << 44), n]
            elif a == "timing":
                c.append(ctypes.byref(timing))
            elif isinstance(a, list) and a[0] == "prob":
                prob = ctypes.create_string_buffer(bytes.fromhex(a[1]), len(a[1]) // 2)
                c.append(prob)
            elif isinstance(a, list):
                c.append(ctypes.c_int32(a[1]))
            else:
                c.append(None if a is None else ctypes.c_double(a) if isinstance(a, float) else ctypes.c_int64(a))
        st = getattr(lib, fn)(*c)
        out.append({"status": st, "ms": list(timing.ms), "counts": list(timing.launches),
                    "launches": [[e.name.decode(), list(e.grid), list(e.block)] for e in launches[:count.value]]})
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _child(*sys.argv[1:])
