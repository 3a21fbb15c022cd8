"""Which summed rotations at N = 8192 take the division by P in the kernel that adds them up, on both sides of the rule's limits, with 256 compute
units.  Runs without a GPU, against a recording stand-in for the runtime."""
import json
import sys

import pytest

from tests.bruteforce import ntt_primes
from tests.stubbed import DEV as d, Stubbed, run, u32, vp
from workloads.params import ParamSet

# log2 N, primes, special primes
SETS = {"k3": (13, 3, 1), "k4": (13, 4, 1), "k6": (13, 6, 1), "k3_p2": (13, 3, 2), "n4096": (12, 2, 1), "n16384": (14, 3, 1)}
# (set, batch, rotations) -> with the mod-down
WANT = {
    # pairs of units, four primes: one round of the special prime's and three of the others' against four
    **{("k3", b, n): False for b in (128, 256, 320, 384, 600, 640, 682) for n in (7, 8)},
    **{("k3", b, n): True for b in (321, 340, 460, 512, 900, 1022, 1024, 1100, 1536) for n in (7, 8)},
    # more rounds only from 1024 units on, with up to three digits and eight rotations
    ("k3", 1100, 9): False, ("k3", 1024, 9): True, ("k3", 1024, 15): True,
    ("k4", 400, 7): False, ("k4", 512, 7): True, ("k4", 1100, 7): False, ("k6", 500, 7): True, ("k6", 600, 7): False,
    ("k3_p2", 512, 7): False, ("n4096", 512, 7): False, ("n16384", 512, 7): False,
}


def _launches(lib):
    got = {}
    gs, keys, out = (u32 * 16)(*range(3, 35, 2)), (vp * 16)(*[1 << 20] * 16), vp(1 << 45)
    for name, (log2n, k, nsp) in SETS.items():
        p = ntt_primes(1 << 50, 2 << log2n, k + nsp)
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
    names = [k[0] for k in launches[" ".join(map(str, case))]]
    if WANT[case]:
        assert [n[:n.index("<")] for n in names] == ["ks_sum_row_kernel", "ks_sum_down_kernel"], names
    else:
        assert names and not any(n.startswith("ks_sum_down") for n in names), names


if __name__ == "__main__":
    print(json.dumps(_launches(Stubbed(*sys.argv[1:]))))
