"""How many launches key switches and products take at batches where a rule of the dispatch changes, with 256 compute units:
the kernels that take a (unit, prime) through several transforms only where enough of their last round is busy.  Runs
without a GPU, against a recording stand-in for the runtime."""
import json
import sys

import pytest

from tests.bruteforce import ntt_primes
from tests.stubbed import DEV as d, Stubbed, run, u32, vp
from workloads.params import ParamSet

SETS = {"n8192_k3": (13, 3), "n4096_k2": (12, 2), "n4096_k3": (12, 3)}
# (set, operation) -> batches by launch: the single transforms' launches, and the kernel that replaces them
WANT = {("n8192_k3", "rotate"): ((32, 36, 42, 65, 96, 129, 140), (43, 48, 64, 97, 128, 141, 193)),
        ("n8192_k3", "relin"): ((31, 32, 65, 95), (33, 36, 64, 96, 129, 193)),
        ("n4096_k2", "rotate"): ((40, 43, 86, 107, 123), (44, 85, 124, 128, 171)),
        ("n4096_k2", "relin"): ((42,), (43, 86, 200)),
        ("n4096_k3", "rotate"): ((32, 42, 65, 90), (43, 64, 93, 129)),
        ("n8192_k3", "sum"): ((38, 41, 65, 102), (42, 64, 107, 193)),
        ("n4096_k2", "sum"): ((42,), (43, 86, 200)),
        ("n4096_k3", "sum"): ((33, 42, 72, 83), (43, 64, 84, 90)),
        ("n8192_k3", "mul"): ((18, 37, 54), (19, 36, 55, 74)),
        ("n4096_k2", "mul"): ((25,), (26, 52, 58)),
        ("n4096_k3", "mul"): ((20, 21, 42, 47), (22, 36, 48, 74)),
        # whole units in one launch instead of rows and the mod-down
        ("n8192_k3", "rotate unit"): ((230, 300, 460, 690), (231, 256, 461, 692)),
        ("n8192_k3", "relin unit"): ((231, 256, 460, 692, 719), (461, 512, 720)),
        ("n4096_k2", "relin unit"): ((256, 460), (461, 692)),
        # rotations of eight ciphertexts (with the mod-up)
        ("n8192_k3", "series"): ((7, 8), (9, 16)),
        ("n4096_k2", "series"): ((7,), (8, 16))}


def _launches(lib):
    got = {}
    for name, (log2n, k) in SETS.items():
        p = ntt_primes(1 << 50, 2 << log2n, k + 1)
        ctx = lib.create(ParamSet(name, log2n, q=tuple(p[:k]), p=tuple(p[k:])))
        gs, keys = (u32 * 16)(*range(3, 35, 2)), (vp * 16)(*[1 << 20] * 16)
        out = vp(1 << 40)        # (an output must not overlap the input)
        calls = {"rotate": lambda b: lib.lib.cg_rotate(ctx, None, d, u32(3), d, out, u32(b), 1, d),
                 "relin": lambda b: lib.lib.cg_relin(ctx, None, d, d, out, u32(b), d),
                 "sum": lambda b: lib.lib.cg_rotate_sum_hoisted(ctx, None, d, u32(3), gs, keys, out, u32(b), d),
                 "series": lambda b: lib.lib.cg_rotate_hoisted(ctx, None, d, u32(b), gs, keys, out, u32(8), d),
                 "mul": lambda b: lib.lib.cg_mul(ctx, None, d, d, out, u32(b), u32(1), d)}
        for (s, op), batches in WANT.items():
            if s == name:
                for b in batches[0] + batches[1]:
                    got[f"{s} {op} {b}"] = len(lib.log(lambda: calls[op.split()[0]](b)))
        assert lib.lib.cg_destroy(ctx) == 0
    return got


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    return run(__file__, tmp_path_factory.mktemp("stub"))


@pytest.mark.parametrize("name,op", WANT, ids=[" ".join(k) for k in WANT])
def test_launches(launches, name, op):
    # with the mod-down or scaling; a product's operands may share one launch instead of two
    apart, together = {"rotate": ({3}, {2}), "relin": ({3}, {2}), "sum": ({4}, {2}), "mul": ({3, 4}, {2}),
                       "rotate unit": ({2}, {1}), "relin unit": ({2}, {1}), "series": ({3}, {2})}[op]
    for b in WANT[name, op][0]:
        assert launches[f"{name} {op} {b}"] in apart, b
    for b in WANT[name, op][1]:
        assert launches[f"{name} {op} {b}"] in together, b


if __name__ == "__main__":
    print(json.dumps(_launches(Stubbed(*sys.argv[1:]))))
