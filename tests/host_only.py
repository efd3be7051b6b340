"""The library on the stand-in of fakehip.c: `load(path of its .so)` in a fresh process,
before anything else loads a HIP runtime.  Kernels do nothing; `calls()` is what the
library asked of the runtime since the last `clear()`."""

import ctypes as C
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))


def build(out):
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-pthread",
                    os.path.join(HERE, "fakehip.c"), "-o", out], check=True)
    return out


def run(so, script, *args):
    """`script` (a file) in a process of its own, with the stand-in's path and `args`."""
    p = subprocess.run([sys.executable, script, so, *args], text=True, capture_output=True,
                       timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr


class Rec(C.Structure):
    _fields_ = [("op", C.c_char * 24), ("name", C.c_char * 72), ("tid", C.c_int64),
                ("stream", C.c_int64), ("a", C.c_int64), ("b", C.c_int64),
                ("bytes", C.c_int64), ("dev", C.c_int64)]


class Call:
    def __init__(self, r):
        self.op, self.name = r.op.decode(), r.name.decode()
        self.tid, self.stream, self.dev = r.tid, r.stream, r.dev
        self.a, self.b, self.bytes = r.a, r.b, r.bytes

    def __repr__(self):
        return f"{self.op}({self.name} stream={self.stream:#x} tid={self.tid} {self.bytes})"


def load(so):
    sys.modules["torch"] = None  # (it would bring a HIP runtime of its own)
    fake = C.CDLL(so, mode=C.RTLD_GLOBAL)
    fake.fake_count.restype = C.c_int64
    fake.fake_in_use.restype = C.c_int64
    fake.fake_record.restype = C.POINTER(Rec)
    fake.fake_record.argtypes = [C.c_int64]
    fake.fake_limit.argtypes = [C.c_int64]
    sys.path.insert(0, os.path.dirname(HERE))
    return fake


def calls(fake):
    return [Call(fake.fake_record(i).contents) for i in range(fake.fake_count())]
