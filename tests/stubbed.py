"""The library's host code without a GPU: loaded behind a recording stand-in for the HIP runtime
(tests/host/hip_runtime_stub.cpp), in a process of its own that must not have loaded the runtime before."""
import ctypes as C
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
vp, u32 = C.c_void_p, C.c_uint32
DEV = vp(1 << 20)                # a device address: passed on, never read


class _Params(C.Structure):
    _fields_ = [("log2n", u32), ("k", u32), ("nsp", u32), ("alpha", u32), ("t", C.c_uint64),
                ("q", C.POINTER(C.c_uint64)), ("p", C.POINTER(C.c_uint64))]


class Stubbed:
    """for the child process"""

    def __init__(self, stub_path, lib_path):
        self.stub = C.CDLL(stub_path, mode=C.RTLD_GLOBAL)
        self.stub.stub_log_size.restype = self.stub.stub_kernel_count.restype = C.c_size_t
        self.stub.stub_log_kernel.restype = self.stub.stub_kernel_name.restype = C.c_char_p
        self.lib = C.CDLL(lib_path)

    def create(self, prm):
        q, p = (C.c_uint64 * prm.k)(*prm.q), (C.c_uint64 * prm.nsp)(*prm.p)
        raw, h = _Params(prm.log2n, prm.k, prm.nsp, prm.alpha, prm.t, q, p), vp()
        assert self.lib.cg_create(C.byref(h), C.byref(raw)) == 0
        return h

    def log(self, call):
        """what `call` (returning a status) does: [(kind, stream, event), ...] as in the stand-in"""
        self.stub.stub_log_clear()
        rc = call()
        assert rc == 0, rc
        out = []
        for i in range(self.stub.stub_log_size()):
            kind, s, e = C.c_int(), vp(), vp()
            self.stub.stub_log_get(C.c_size_t(i), C.byref(kind), C.byref(s), C.byref(e))
            out.append((kind.value, s.value or 0, e.value or 0))
        return out


    def kernels(self, call):
        """the kernels `call` launches: [[name with its template arguments, blocks, threads], ...]"""
        out = []
        for i in range(len(self.log(call))):
            blocks, threads = u32(), u32()
            name = self.stub.stub_log_kernel(C.c_size_t(i), C.byref(blocks), C.byref(threads)).decode()
            if name:
                out.append([short(name), blocks.value, threads.value])
        return out

    def compiled(self):
        """every kernel of the library"""
        return [short(self.stub.stub_kernel_name(C.c_size_t(i)).decode()) for i in range(self.stub.stub_kernel_count())]


def short(name):
    """void cg::scale_kernel<2, false>(...) -> scale_kernel<2, false>"""
    depth = 0
    for i, ch in enumerate(name):
        depth += {"<": 1, ">": -1}.get(ch, 0)
        if ch == "(" and not depth:
            name = name[:i]
            break
    return name.removeprefix("void ").replace("cg::", "")


def run(script, tmp):
    """runs a test module as the child: its main gets a Stubbed and prints JSON, which this returns"""
    from paper_2602_08798_amd import binding
    so = os.path.join(str(tmp), "stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so,
                    os.path.join(ROOT, "tests", "host", "hip_runtime_stub.cpp")], check=True)
    child = subprocess.run([sys.executable, os.path.abspath(script), so, binding._LIB_PATH], capture_output=True,
                           text=True, cwd=ROOT, env={**os.environ, "PYTHONPATH": ROOT})
    assert child.returncode == 0, child.stderr
    return json.loads(child.stdout)
