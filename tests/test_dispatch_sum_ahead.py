"""Which summed inner products from digits in memory ask for their words a rotation ahead, on both sides of the rule's limits, with 256 compute
units.  Runs without a GPU, against a recording stand-in for the runtime."""
import json
import sys

import pytest

from tests.bruteforce import ntt_primes
from tests.stubbed import DEV as d, Stubbed, run, u32, vp
from workloads.params import ParamSet

# log2 N, primes (a digit each)
SETS = {"k1": (13, 1), "k2": (13, 2), "k3": (13, 3), "k4": (13, 4), "k6": (13, 6), "n4096": (12, 2), "n16384": (14, 3)}
# (set, batch, rotations) -> ciphertexts per thread, ahead
WANT = {
    # one rotation has none to look ahead to
    **{(s, 1, 1): (1, False) for s in SETS}, ("k3", 12, 1): (2, False), ("n4096", 42, 1): (2, False),
    # N = 8192, more than one workgroup per compute unit: keys of a prime below 7/8 of an XCD's L2 (three digits: nine rotations)
    **{("k3", b, n): (1, True) for b in (3, 6, 10) for n in (2, 7, 9)}, **{("k3", b, n): (1, False) for b in (3, 6, 10) for n in (10, 15, 31)},
    **{("k3", b, n): (2, True) for b in (12, 20) for n in (2, 9)}, **{("k3", b, n): (2, False) for b in (12, 20) for n in (10, 15)},
    ("k2", 12, 13): (1, True), ("k2", 12, 14): (1, False), ("k4", 12, 6): (2, True), ("k4", 12, 7): (2, False), ("k1", 16, 63): (1, True),
    # up to one workgroup: always
    **{("k3", b, 31): (1, True) for b in (1, 2)}, ("k4", 1, 31): (1, True), ("k4", 2, 31): (1, False),
    # five and six digits: not with one a thread
    ("k6", 6, 7): (1, False), ("k6", 12, 15): (2, True),
    ("n4096", 24, 31): (1, True), ("n4096", 42, 31): (2, True), ("n16384", 2, 31): (1, True),
    # four and eight a thread never
    ("k3", 24, 7): (4, False), ("k3", 36, 3): (4, False),
}


def _launches(lib):
    got = {}
    gs, keys, out = (u32 * 64)(*range(3, 131, 2)), (vp * 64)(*[1 << 20] * 64), vp(1 << 45)
    for name, (log2n, k) in SETS.items():
        p = ntt_primes(1 << 50, 2 << log2n, k + 1)
        ctx = lib.create(ParamSet(name, log2n, q=tuple(p[:k]), p=tuple(p[k:]), alpha=1))
        for s, batch, n in WANT:
            if s == name:
                got[f"{s} {batch} {n}"] = lib.kernels(lambda: lib.lib.cg_rotate_sum_hoisted(ctx, None, d, u32(n), gs, keys, out, u32(batch), d))
        assert lib.lib.cg_destroy(ctx) == 0
    return got


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    return run(__file__, tmp_path_factory.mktemp("stub"))


@pytest.mark.parametrize("case", WANT, ids=lambda c: " ".join(map(str, c)))
def test_route(launches, case):
    per_thread, ahead = WANT[case]
    names = [k[0] for k in launches[" ".join(map(str, case))]]
    assert f"ks_sum_kernel<{SETS[case[0]][1]}, {per_thread}, {str(ahead).lower()}>" in names, names


if __name__ == "__main__":
    print(json.dumps(_launches(Stubbed(*sys.argv[1:]))))
