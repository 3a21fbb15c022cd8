"""Which kernel a call takes, and how wide, on both sides of the limits that a count of launches does not show, with 256 compute
units.  Runs without a GPU, against a recording stand-in for the runtime."""
import json
import sys

import pytest

from tests.bruteforce import ntt_primes
from tests.stubbed import DEV as d, Stubbed, run, u32, vp
from workloads.params import ParamSet

# name -> log2 N, primes, special primes, primes of a digit
SETS = {"n16384_k6": (14, 6, 2, 2)}
# set, call, its sizes -> the kernel among its launches that tells the routes apart
WANT = {
    # a transformed cache at N = 16384: parts of one unit each (the fewest that are as fast), and of several
    **{("n16384_k6", "context_ext", h, c): "mul_row_kernel<13, 8, 0, true>" for h, c in ((1, 1), (1, 4), (2, 4), (3, 2), (16, 1))},
    **{("n16384_k6", "context_ext", h, c): "mul_sum_row_kernel<13, 8, 0, true>" for h, c in ((4, 4), (8, 3), (12, 2), (16, 3))},
}


def _launches(lib):
    got = {}
    gs, keys, out = (u32 * 16)(*range(3, 35, 2)), (vp * 64)(*[1 << 20] * 64), vp(1 << 40)   # (no output overlaps its input)
    for name, (log2n, k, nsp, alpha) in SETS.items():
        p = ntt_primes(1 << 50, 2 << log2n, k + nsp)
        ctx = lib.create(ParamSet(name, log2n, q=tuple(p[:k]), p=tuple(p[k:]), alpha=alpha))
        calls = {"context_ext": lambda h, c: lib.lib.cg_decode_context_hoisted(
            ctx, None, d, d, d, u32(h), u32(c), u32(c), u32(64), u32(3), 1, d, keys, out, d)}
        for (s, op, *sizes), _ in WANT.items():
            if s == name:
                got[" ".join(map(str, (s, op, *sizes)))] = lib.kernels(lambda: calls[op](*sizes))
        assert lib.lib.cg_destroy(ctx) == 0
    return got


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    return run(__file__, tmp_path_factory.mktemp("stub"))


@pytest.mark.parametrize("case", WANT, ids=lambda c: " ".join(map(str, c)))
def test_kernel(launches, case):
    names = [k[0] for k in launches[" ".join(map(str, case))]]
    assert WANT[case] in names, names


if __name__ == "__main__":
    print(json.dumps(_launches(Stubbed(*sys.argv[1:]))))
