"""Which streams the one-call decode step puts its branches on, and what they wait for.  Runs without a GPU: the library's
host code against a recording stand-in for the runtime (tests/host/hip_runtime_stub.cpp), in a process of its own."""
import ctypes as C
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
S1, S2 = 0x1000, 0x2000          # callers' streams (never dereferenced)


def _record(stub_path, lib_path):
    """steps of two contexts on several streams -> {name: [(kind, stream, event), ...]}"""
    stub = C.CDLL(stub_path, mode=C.RTLD_GLOBAL)
    stub.stub_log_size.restype = C.c_size_t
    lib = C.CDLL(lib_path)
    vp, u32 = C.c_void_p, C.c_uint32

    class Params(C.Structure):
        _fields_ = [("log2n", u32), ("k", u32), ("nsp", u32), ("alpha", u32), ("t", C.c_uint64),
                    ("q", C.POINTER(C.c_uint64)), ("p", C.POINTER(C.c_uint64))]

    from workloads import PRESETS
    prm = PRESETS["C1"]
    q, p = (C.c_uint64 * prm.k)(*prm.q), (C.c_uint64 * prm.nsp)(*prm.p)
    raw = Params(prm.log2n, prm.k, prm.nsp, prm.alpha, prm.t, q, p)
    ctx = []
    for _ in range(2):
        h = vp()
        assert lib.cg_create(C.byref(h), C.byref(raw)) == 0
        ctx.append(h)
    d = vp(1 << 20)              # a device address: passed on, never read
    keys = (vp * 64)(*[1 << 20] * 64)
    d2, blocks = 64, prm.n // 64

    def step(c, stream, opens, hoisted):
        heads, n_cts, stride = 2, 1, 2
        tau = blocks if opens else blocks - 1
        stub.stub_log_clear()
        common = [ctx[c], vp(stream), d, d, d]
        geometry = [u32(heads), u32(n_cts), u32(stride), u32(d2), u32(tau), d, d, d]
        if hoisted:
            rc = lib.cg_decode_step_hoisted(*common, d, *geometry, u32(3), keys, u32(3), 1, keys, d, d, d)
        else:
            rc = lib.cg_decode_step(*common, *geometry, keys, keys, d, d, d)
        assert rc == 0, rc
        out = []
        for i in range(stub.stub_log_size()):
            kind, s, e = C.c_int(), vp(), vp()
            stub.stub_log_get(C.c_size_t(i), C.byref(kind), C.byref(s), C.byref(e))
            out.append((kind.value, s.value or 0, e.value or 0))
        return out

    got = {}
    for c in range(2):
        for stream in (0, S1, S2):
            for opens in (False, True):
                for hoisted in (False, True):
                    got[f"{c},{stream},{int(opens)},{int(hoisted)}"] = step(c, stream, opens, hoisted)
    for h in ctx:
        assert lib.cg_destroy(h) == 0
    return got


@pytest.fixture(scope="module")
def log(tmp_path_factory):
    from paper_2602_08798_amd import binding
    so = str(tmp_path_factory.mktemp("stub") / "stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so,
                    os.path.join(ROOT, "tests", "host", "hip_runtime_stub.cpp")], check=True)
    run = subprocess.run([sys.executable, os.path.abspath(__file__), so, binding._LIB_PATH], capture_output=True,
                         text=True, cwd=ROOT, env={**os.environ, "PYTHONPATH": ROOT})
    assert run.returncode == 0, run.stderr
    return {tuple(int(v) for v in k.split(",")): [tuple(e) for e in v] for k, v in json.loads(run.stdout).items()}


def _streams(entries, but=None):
    return {s for _, s, _ in entries} - {but}


def test_steps_of_two_contexts_on_two_streams_share_no_stream(log):
    """what one caller's stream waits for must never hold up a step that another caller issues elsewhere"""
    for opens in (0, 1):
        for hoisted in (0, 1):
            for a, b in ((S1, S2), (0, S1), (S1, 0)):
                assert not _streams(log[0, a, opens, hoisted]) & _streams(log[1, b, opens, hoisted]), (a, b)


def test_steps_on_the_default_stream_use_one_pair(log):
    """(with a pair per context the pairs of later contexts come to lie on the caller's own hardware queue)"""
    for opens in (0, 1):
        assert _streams(log[0, 0, opens, 1], 0) == _streams(log[1, 0, opens, 1], 0)
        assert len(_streams(log[0, 0, opens, 1], 0)) == 1 + opens


def test_branches_fork_from_and_join_the_callers_stream(log):
    for (_, stream, opens, _), entries in log.items():
        recorded = {}            # event -> (stream, position) of its last record
        first_wait, last_work, joined = {}, {}, set()
        for i, (kind, s, e) in enumerate(entries):
            if kind == 1:
                recorded[e] = (s, i)
            elif kind == 2 and s != stream:
                assert recorded[e][0] == stream
                first_wait.setdefault(s, i)
            elif kind == 2:
                side, at = recorded[e]
                assert last_work[side] < at
                joined.add(side)
            else:
                assert s == stream or s in first_wait, "work on a side stream before it waited for the fork"
                last_work[s] = i
        assert joined == _streams(entries, stream)
        assert all(i < entries.index(next(x for x in entries if x[0] == 2 and x[1] == stream)) for s, i in
                   last_work.items() if s != stream)


if __name__ == "__main__":
    print(json.dumps(_record(sys.argv[1], sys.argv[2])))
