"""Products at N = 16384, where operands are lifted ahead and the two halves of a row are transformed apart: every number of
primes, primes of different sizes, half rows below and above the number of compute units (2 (2k + 1) of them per product, 256
units), shared operands with a ragged last group, and sums in parts.  Bit-compared with the oracle; units repeat a few
distinct operands, extreme residues among them, so that every unit is checked."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads import PRESETS
from workloads.params import ParamSet

from .bruteforce import ntt_primes
from .test_gpu_parity import Env, say
from .test_gpu_row_kernels import _extremes, _tiled


def _set(k, nsp, alpha):
    p = ntt_primes(1 << 50, 2 << 14, k + nsp)
    return ParamSet(f"n16384_k{k}", 14, q=tuple(p[:k]), p=tuple(p[k:]), alpha=alpha)


SETS = {"k1": _set(1, 1, 1), "k2": _set(2, 1, 1), "k4": _set(4, 2, 2), "k5": _set(5, 2, 1), "C5": PRESETS["C5"],
        "mixed": ParamSet("mixed_n16384_k3", 14, q=tuple(p for b in (50, 43, 48) for p in ntt_primes(1 << b, 2 << 14, 1)),
                          p=tuple(ntt_primes((1 << 50) - (1 << 45), 2 << 14, 1)), alpha=1)}
_envs = {}


def _env(name):
    if name not in _envs:
        import paper_2602_08798_amd as P
        from oracle import Oracle
        env, prm = Env.__new__(Env), SETS[name]
        env.P, env.name, env.prm, env.ctx, env.orc = P, name, prm, P.Context(prm), Oracle(prm)
        env.n, env.k, env.qp, env._keys = prm.n, prm.k, list(prm.q) + list(prm.p), {}
        _envs[name] = env
    return _envs[name]


@pytest.mark.parametrize("name,batches", [("k1", (1, 42, 43)), ("k2", (26,)), ("k4", (14, 15)), ("k5", (1, 12)),
                                          ("C5", (9, 10, 21)), ("mixed", (18, 19, 40))])
def test_products(name, batches):
    env = _env(name)
    a, b = _extremes(env, env.cts(10, 3)), _extremes(env, env.cts(11, 2))
    want = {(i, j): env.orc.mul(a[i], b[j]) for i in range(3) for j in range(2)}
    for batch in batches:
        say(f"mul {name} batch {batch}")
        got = env.host(env.ctx.mul(_tiled(env, a, batch), _tiled(env, b, batch), batch))
        for u in range(batch):
            assert np.array_equal(got[u], want[u % 3, u % 2]), (name, batch, u)
    for batch, group in ((5, 2), (12, 5)):
        say(f"mul {name} batch {batch}, a operands shared by {group}")
        got = env.host(env.ctx.mul(_tiled(env, a, -(-batch // group)), _tiled(env, b, batch), batch, a_group=group))
        for u in range(batch):
            assert np.array_equal(got[u], want[u // group % 3, u % 2]), (name, batch, group, u)


@pytest.mark.parametrize("name,shapes", [("C5", ((1, 1), (1, 24), (10, 2))), ("k1", ((1, 70), (44, 2))), ("mixed", ((3, 7),))])
def test_sums_of_products_in_parts(name, shapes):
    env = _env(name)
    a, b = _extremes(env, env.cts(14, 3)), _extremes(env, env.cts(15, 2))
    for groups, group in shapes:
        say(f"mul_sum {name}: {groups} groups of {group}")
        n = groups * group
        got = env.host(env.ctx.mul_sum(_tiled(env, a, n), _tiled(env, b, n), groups, group))
        want = {}
        for g in range(groups):
            key = (g * group) % 6
            if key not in want:
                us = range(g * group, (g + 1) * group)
                want[key] = env.orc.mul_sum([a[u % 3] for u in us], [b[u % 2] for u in us])
            assert np.array_equal(got[g], want[key]), (name, groups, group, g)
