"""Which kernel a call takes, and how wide, on both sides of the limits that a count of launches does not show, with 256 compute
units.  Runs without a GPU, against a recording stand-in for the runtime."""
import ctypes as C
import json
import sys

import pytest

from tests.bruteforce import ntt_primes
from tests.stubbed import DEV as d, Stubbed, run, u32, vp
from workloads.params import ParamSet

class _KernelStat(C.Structure):
    _fields_ = [("kernel_id", u32), ("launches", u32), ("total_ms", C.c_double), ("algo_bytes", C.c_double),
                ("work_items", C.c_double)]


# name -> log2 N, primes, special primes, primes of a digit
SETS = {"n8192_k3": (13, 3, 1, 1), "n16384_k6": (14, 6, 2, 2)}
# set, call, its sizes -> the kernel among its launches that tells the routes apart
WANT = {
    # a transformed cache at N = 16384: parts of one unit each (the fewest that are as fast), and of several
    **{("n16384_k6", "context_ext", h, c): "mul_row_kernel<13, 8, 0, true>" for h, c in ((1, 1), (1, 4), (2, 4), (3, 2), (16, 1))},
    **{("n16384_k6", "context_ext", h, c): "mul_sum_row_kernel<13, 8, 0, true>" for h, c in ((4, 4), (8, 3), (12, 2), (16, 3))},
}


def _profile(lib, ctx, call):
    """kernel classes the library's own timing names for `call`: [[name, launches, items], ...]"""
    stats, n = (_KernelStat * 64)(), u32()
    lib.lib.cg_kernel_name.restype = C.c_char_p
    assert lib.lib.cg_profile_begin(ctx, u32(256)) == 0
    assert call() == 0
    assert lib.lib.cg_profile_end(ctx, stats, u32(64), C.byref(n)) == 0
    return [[lib.lib.cg_kernel_name(s.kernel_id).decode(), s.launches, s.work_items] for s in stats[:n.value]]


def _launches(lib):
    got = {}
    gs, keys, out = (u32 * 16)(*range(3, 35, 2)), (vp * 256)(*[1 << 20] * 256), vp(1 << 40)   # (no output overlaps its input)
    for name, (log2n, k, nsp, alpha) in SETS.items():
        p = ntt_primes(1 << 50, 2 << log2n, k + nsp)
        ctx = lib.create(ParamSet(name, log2n, q=tuple(p[:k]), p=tuple(p[k:]), alpha=alpha))
        calls = {"context_ext": lambda h, c: lib.lib.cg_decode_context_hoisted(
            ctx, None, d, d, d, u32(h), u32(c), u32(c), u32(64), u32(3), 1, d, keys, out, d)}
        for (s, op, *sizes), _ in WANT.items():
            if s == name:
                got[" ".join(map(str, (s, op, *sizes)))] = lib.kernels(lambda: calls[op](*sizes))
        if name == "n8192_k3":
            got["profile"] = _profile(lib, ctx, lambda: lib.lib.cg_prefill_av_hoisted(ctx, None, d, d, u32(3), u32(64), 1, d, keys,
                                                                                      out, d))
        assert lib.lib.cg_destroy(ctx) == 0
    return got


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    return run(__file__, tmp_path_factory.mktemp("stub"))


@pytest.mark.parametrize("case", WANT, ids=lambda c: " ".join(map(str, c)))
def test_kernel(launches, case):
    names = [k[0] for k in launches[" ".join(map(str, case))]]
    assert WANT[case] in names, names


def test_copies_are_not_timed_as_sums(launches):
    """A V of three heads: a copy of every head's V, rotated copies, products, one relinearisation; nothing is added up"""
    classes = {name: (n, items) for name, n, items in launches["profile"]}
    assert classes["copy"] == (1, 3)
    assert "add" not in classes


if __name__ == "__main__":
    print(json.dumps(_launches(Stubbed(*sys.argv[1:]))))
