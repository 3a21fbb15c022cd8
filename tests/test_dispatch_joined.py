"""Which chains of single rotations and which rounds of summed rotations take the mod-down before them in the mod-up's loader, on both sides of the rules'
limits, in calls made alone and in steps, with 256 compute units; and where callers' inverse transforms go over to 512 threads.  Runs without a
GPU, against a recording stand-in for the runtime."""
import json
import sys

import pytest

from tests.bruteforce import ntt_primes
from tests.stubbed import DEV as d, Stubbed, run, u32, vp
from workloads.params import ParamSet

# log2 N, primes (a digit each)
SETS = {"k1": (13, 1), "k2": (13, 2), "k3": (13, 3), "k4": (13, 4), "n4096_k1": (12, 1), "n4096_k2": (12, 2), "n4096_k3": (12, 3)}
# (set, call, its sizes) -> key switches that take the mod-down before them; a chain has a switch for every bit of d2 (scores) or N/d2 (context)
CHAINS = {
    # scores alone, units, d2: the mod-up's rows and the launch behind it
    **{("k3", "scores", u, 64): n for u, n in ((1, 6), (21, 6), (22, 0))}, **{("k2", "scores", u, 64): n for u, n in ((34, 6), (35, 0))},
    **{("k1", "scores", u, 64): n for u, n in ((64, 6), (65, 0))}, ("k4", "scores", 1, 64): 0,
    **{("n4096_k2", "scores", u, 64): n for u, n in ((64, 6), (65, 0))}, **{("n4096_k1", "scores", u, 64): n for u, n in ((117, 6), (118, 0))},
    **{("n4096_k3", "scores", u, 64): n for u, n in ((32, 6), (33, 0))}, **{("n4096_k2", "scores", u, 2): n for u, n in ((43, 1), (44, 0))},
    # steps, heads x ciphertexts, d2 (64: scores 6, context 7 at N = 8192 and 6 at N = 4096)
    **{("k3", "step", *s, 64): n for s, n in (((1, 1), 13), ((7, 3), 13), ((11, 2), 0), ((8, 3), 0), ((22, 1), 0))},
    # ... a context with two switches less or more to do than the scores (32: scores 5, context 8), beside a mod-up row for every unit
    **{("k3", "step", *s, 32): n for s, n in (((12, 4), 8), ((21, 3), 8), ((12, 5), 8), ((13, 5), 0), ((10, 3), 8))},
    # ... the scores beside a context with a mod-up row for every unit
    **{("n4096_k2", "step", *s, 64): n for s, n in (((42, 1), 12), ((43, 1), 0), ((16, 4), 6), ((10, 4), 12))},
    # ... other numbers of digits: fewer units
    **{("k1", "step", *s, 64): n for s, n in (((48, 1), 13), ((49, 1), 0))}, **{("k2", "step", *s, 64): n for s, n in (((26, 1), 13), ((27, 1), 0))},
    **{("n4096_k3", "step", *s, 64): n for s, n in (((18, 1), 12), ((19, 1), 0))},
}
# rounds: of the scores, of the context
ROUNDS = {
    **{("k3", "scores", u, 64, 3): n for u, n in ((3, 2), (4, 0))}, **{("k1", "scores", u, 64, 3): n for u, n in ((8, 2), (9, 0))},
    **{("k2", "scores", u, 64, 3): n for u, n in ((4, 2), (5, 0))}, **{("n4096_k2", "scores", u, 64, 3): n for u, n in ((21, 2), (22, 0))},
    **{("n4096_k1", "scores", u, 64, 3): n for u, n in ((37, 2), (38, 0))}, **{("n4096_k3", "scores", u, 64, 3): n for u, n in ((10, 2), (11, 0))},
    # rounds of 15 rotations, alone: one workgroup of the sums to a unit
    **{("k3", "context", u, 64, 4): n for u, n in ((2, 2), (3, 0))},
    # steps at d2 = 64, N = 8192: scores 2 rounds, context 3; beside the scores' mod-ups for 3/8 of the units
    **{("k3", "step", *s, 64, 3): n for s, n in (((1, 1), 5), ((5, 1), 5), ((6, 1), 0), ((1, 5), 5), ((1, 6), 3), ((1, 8), 3), ((1, 9), 0), ((4, 2), 3), ((3, 3), 0))},
    # ... d2 = 128: scores 3, context 2, which is not joined beside longer scores of more than a quarter
    **{("k3", "step", *s, 128, 3): n for s, n in (((5, 1), 5), ((1, 5), 5), ((2, 3), 0), ((4, 2), 0))},
    # ... rounds of 15 rotations in either branch: up to three units
    **{("k3", "step", *s, 64, 4): n for s, n in (((3, 1), 4), ((4, 1), 0), ((3, 2), 2), ((1, 3), 4), ((1, 4), 2))},
    **{("k3", "step", *s, 256, 4): n for s, n in (((3, 1), 4), ((4, 1), 0))},
    **{("k1", "step", *s, 64, 3): n for s, n in (((13, 1), 5), ((14, 1), 0))}, **{("k2", "step", *s, 64, 3): n for s, n in (((8, 1), 5), ((9, 1), 0))},
    # ... N = 4096: both branches' mod-ups for 7/8 of the units
    **{("n4096_k2", "step", *s, 64, 3): n for s, n in (((18, 1), 4), ((19, 1), 0), ((12, 2), 2), ((13, 2), 0), ((9, 3), 2), ((10, 3), 0))},
}
# the first mod-up of a chain of up to half a row per unit in parts, but beside a mod-up row for every unit of the other branch
PARTS = {("k3", "context", 10, 64): True, ("k3", "step", 10, 3, 32): False, ("k3", "step", 4, 8, 32): False, ("k3", "step", 7, 3, 64): True}
INVERSE = {("k3", 384): 8, ("k3", 385): 16, ("k3", 16384): 16}      # rows -> elements per thread


def _launches(lib):
    got = {}
    keys, out = (vp * 256)(*[1 << 20] * 256), vp(1 << 45)       # (no output overlaps its input)
    f, b = lib.lib, lambda *x: [u32(v) for v in x]
    for name, (log2n, k) in SETS.items():
        p = ntt_primes(1 << 50, 2 << log2n, k + 1)
        ctx = lib.create(ParamSet(name, log2n, q=tuple(p[:k]), p=tuple(p[k:]), alpha=1))
        tau = lambda c, d2: u32(c * (1 << log2n) // d2 - 1)
        calls = {"scores": lambda u, d2, w=0: f.cg_decode_scores_hoisted(ctx, None, d, d, None, *b(u, 1, 1, d2, w), d, keys, out, d) if w else
                           f.cg_decode_scores(ctx, None, d, d, *b(u, 1, 1, d2), d, keys, out, d),
                 "context": lambda u, d2, w=0: f.cg_decode_context_hoisted(ctx, None, d, d, None, *b(u, 1, 1, d2, w, 1), d, keys, out, d) if w else
                            f.cg_decode_context(ctx, None, d, d, *b(u, 1, 1, d2), d, keys, out, d),
                 "step": lambda h, c, d2, w=0: f.cg_decode_step_hoisted(ctx, None, d, d, d, None, *b(h, c, c + 1, d2), tau(c, d2), d, d, d, u32(w), keys, u32(w), 1,
                                                                        keys, out, out, d) if w else
                         f.cg_decode_step(ctx, None, d, d, d, *b(h, c, c + 1, d2), tau(c, d2), d, d, d, keys, keys, out, out, d)}
        for s, op, *sizes in [*CHAINS, *ROUNDS, *PARTS]:
            if s == name:
                got[" ".join(map(str, (s, op, *sizes)))] = lib.kernels(lambda: calls[op](*sizes))
        for s, rows in INVERSE:
            if s == name:
                got[f"{s} {rows}"] = lib.kernels(lambda: f.cg_ntt_inverse(ctx, None, d, out, (u32 * rows)(*[i % k for i in range(rows)]), u32(rows)))
        assert f.cg_destroy(ctx) == 0
    return got


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    return run(__file__, tmp_path_factory.mktemp("stub"))


def _count(launches, case, kernel):
    names = [k[0] for k in launches[" ".join(map(str, case))]]
    assert names
    return sum(n.startswith(kernel) for n in names)


@pytest.mark.parametrize("case", CHAINS, ids=lambda c: " ".join(map(str, c)))
def test_chains(launches, case):
    assert _count(launches, case, "ks_inner_after_kernel<") == CHAINS[case]


@pytest.mark.parametrize("case", ROUNDS, ids=lambda c: " ".join(map(str, c)))
def test_rounds(launches, case):
    assert _count(launches, case, "ks_sum_after_kernel<") == ROUNDS[case]


@pytest.mark.parametrize("case", PARTS, ids=lambda c: " ".join(map(str, c)))
def test_first_mod_up(launches, case):
    assert _count(launches, case, "ks_inner_after_kernel<")
    assert bool(_count(launches, case, "ntt_fwd_part_kernel<13, 1, LdModup<false, 1>")) == PARTS[case]


@pytest.mark.parametrize("case", INVERSE, ids=lambda c: " ".join(map(str, c)))
def test_inverse_rows(launches, case):
    assert _count(launches, case, f"ntt_inv_kernel<13, {INVERSE[case]}, LdInvU64, StInvU64>") == 1


if __name__ == "__main__":
    print(json.dumps(_launches(Stubbed(*sys.argv[1:]))))
