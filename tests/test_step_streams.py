"""Which streams the one-call decode step puts its branches on, and what they wait for.  Runs without a GPU: the library's
host code against a recording stand-in for the runtime."""
import ctypes as C
import json
import sys

import pytest

from tests.stubbed import DEV as d, Stubbed, run, u32, vp

S1, S2 = 0x1000, 0x2000          # callers' streams (never dereferenced)


def _record(lib):
    """steps of two contexts on several streams -> {name: [(kind, stream, event), ...]}"""
    from workloads import PRESETS
    prm = PRESETS["C1"]
    ctx = [lib.create(prm) for _ in range(2)]
    keys = (vp * 64)(*[1 << 20] * 64)
    d2, blocks = 64, prm.n // 64

    def step(c, stream, opens, hoisted):
        heads, n_cts, stride = 2, 1, 2
        tau = blocks if opens else blocks - 1
        common = [ctx[c], vp(stream), d, d, d]
        geometry = [u32(heads), u32(n_cts), u32(stride), u32(d2), u32(tau), d, d, d]
        if hoisted:
            return lib.lib.cg_decode_step_hoisted(*common, d, *geometry, u32(3), keys, u32(3), 1, keys, d, d, d)
        return lib.lib.cg_decode_step(*common, *geometry, keys, keys, d, d, d)

    got = {f"{c},{stream},{int(opens)},{int(hoisted)}": lib.log(lambda: step(c, stream, opens, hoisted))
           for c in range(2) for stream in (0, S1, S2) for opens in (False, True) for hoisted in (False, True)}
    for h in ctx:
        assert lib.lib.cg_destroy(h) == 0
    got["context first"] = _context_first(lib)
    return got


# heads x ciphertexts at N = 8192 -> the context on the caller's stream: few rows of the scores (units x 4 primes, up to half of 256 compute units), or these in
# one round and with the context's mod-ups (heads x 12 rows) 5/4 of the units
ORDER = {True: ((4, 4), (16, 2), (8, 7), (8, 8), (9, 6), (10, 5), (12, 4), (14, 3), (16, 4)),
         False: ((3, 11), (11, 3), (11, 4), (9, 5), (8, 6), (6, 8), (13, 3), (9, 8), (11, 6), (13, 5))}
# ... while the context has more key switches one after the other: parameters, heads, ciphertexts, d2, bits of a round -> whether it has
LONGER = {("C2", 6, 3, 64, 3): True, ("C2", 6, 3, 64, 4): False, ("C2", 6, 3, 128, 3): False, ("C2", 12, 4, 64, 4): False, ("C5", 3, 3, 64, 3): True,
          ("C5", 3, 3, 128, 3): False, ("C1", 4, 4, 64, 3): True, ("C1", 4, 4, 128, 3): False}


def _context_first(lib):
    from workloads import PRESETS
    keys, got = (vp * 64)(*[1 << 20] * 64), []
    ctx = {name: lib.create(PRESETS[name]) for name in ("C1", "C2", "C5")}
    for name, h, c, d2, bits in [("C2", h, c, 64, 3) for h, c in ORDER[True] + ORDER[False]] + list(LONGER):
        entries = lib.log(lambda: lib.lib.cg_decode_step_hoisted(
            ctx[name], vp(S1), d, d, d, None, u32(h), u32(c), u32(c), u32(d2), u32(c * PRESETS[name].n // d2 - 1), d, d, d, u32(bits), keys, u32(bits), 1,
            keys, d, d, d))
        scaled = {}                  # blocks of a scaling (more with more results) -> stream
        for i, (_, stream, _) in enumerate(entries):
            blocks, threads = u32(), u32()
            if b"scale_kernel" in lib.stub.stub_log_kernel(C.c_size_t(i), C.byref(blocks), C.byref(threads)):
                scaled[blocks.value] = stream
        got.append([[name, h, c, d2, bits], scaled[min(scaled)] == S1 and scaled[max(scaled)] != S1])
    for h in ctx.values():
        assert lib.lib.cg_destroy(h) == 0
    return got


@pytest.fixture(scope="module")
def recorded(tmp_path_factory):
    return run(__file__, tmp_path_factory.mktemp("stub"))


@pytest.fixture(scope="module")
def log(recorded):
    got = {k: v for k, v in recorded.items() if k != "context first"}
    return {tuple(int(v) for v in k.split(",")): [tuple(e) for e in v] for k, v in got.items()}


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


def test_which_branch_runs_on_the_callers_stream(recorded):
    want = {**{("C2", *shape, 64, 3): first for first in ORDER for shape in ORDER[first]}, **LONGER}
    assert {tuple(case): first for case, first in recorded["context first"]} == want


if __name__ == "__main__":
    print(json.dumps(_record(Stubbed(*sys.argv[1:]))))
