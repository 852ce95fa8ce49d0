"""Host-side tests without a GPU: the library on a HIP runtime in host memory
(host_hip.c; not collected by pytest).

`run(module, case, **kw)` calls module.case(hh, gsp, **kw) in a process of its
own, where libgsp.so allocates host memory and its kernels are written to a
log instead of being run.  What a kernel would be given, and whether it fits
the allocation it points into, can be read from the log."""
import ctypes as C
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host_hip.c")


class Launch(C.Structure):
    _fields_ = [("name", C.c_char * 160), ("grid", C.c_uint32 * 3), ("block", C.c_uint32 * 3), ("lds", C.c_uint64),
                ("arg", C.c_ubyte * 400), ("replayed", C.c_int32), ("pad", C.c_int32)]


class HostHip:
    def __init__(self, path):
        # before torch and libgsp.so, so that both bind to it
        self.lib = lib = C.CDLL(path, mode=C.RTLD_GLOBAL)
        lib.hh_log.restype = C.POINTER(Launch)
        lib.hh_room.restype = C.c_int64
        lib.hh_room.argtypes = [C.c_uint64]
        lib.hh_used.restype = C.c_uint64
        lib.hh_limit.argtypes = [C.c_uint64]

    def launches(self, part=""):
        """The log's launches whose kernel name holds `part`."""
        out = []
        for k in range(self.lib.hh_log_size()):
            l = self.lib.hh_log(k).contents
            if part in l.name.decode():
                out.append(l)
        return out

    def clear(self):
        self.lib.hh_log_clear()

    def limit(self, nbytes):
        self.lib.hh_limit(nbytes)

    def used(self):
        return int(self.lib.hh_used())

    def room(self, p):
        return int(self.lib.hh_room(p))

    def malloc(self, nbytes):
        p = C.c_void_p()
        assert self.lib.hipMalloc(C.byref(p), C.c_size_t(nbytes)) == 0
        return p


def build(folder) -> str:
    so = os.path.join(str(folder), "libhost_hip.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-std=gnu11", "-o", so, SRC, "-lpthread"])
    return so


def run(so, module, case, timeout=300, **kw):
    r = subprocess.run([sys.executable, "-m", "tests.host_hip", so, module, case, json.dumps(kw)], cwd=ROOT,
                       capture_output=True, text=True, timeout=timeout)
    sys.stdout.write(r.stdout[-4000:])
    assert r.returncode == 0, r.stderr[-4000:]


if __name__ == "__main__":
    hh = HostHip(sys.argv[1])
    import importlib
    from paper_2110_12749_amd import gsp
    getattr(importlib.import_module(sys.argv[2]), sys.argv[3])(hh, gsp, **json.loads(sys.argv[4]))
