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


# parts of one unit each (1 x 1, 3 x 2 and, one prime, 1 x 5), of several (44 x 2, 14 x 3, 10 x 2: a whole group), of several and
# uneven (3 x 7, 1 x 70, 1 x 24)
@pytest.mark.parametrize("name,shapes", [("k1", ((1, 5), (1, 70), (44, 2))), ("k4", ((1, 1), (14, 3))),
                                         ("C5", ((3, 2), (10, 2), (1, 24))), ("mixed", ((3, 7),))])
def test_context_sums_with_a_transformed_copy(name, shapes):
    from oracle import attention
    env = _env(name)
    d2 = env.n // 4
    raw_rlk, rlk = env.key(80)
    gs = env.ctx.round_galois(1, d2, 1)
    raws, keys = zip(*[env.key(81 + i) for i in range(len(gs))])
    a, vc = _extremes(env, env.cts(90, 3)), _extremes(env, env.cts(91, 2))
    for heads, n_cts in shapes:
        say(f"decode_context_hoisted {name}: {heads} heads of {n_cts} ciphertexts, transformed copy")
        n = heads * n_cts
        ext = env.ctx.cache_extend(_tiled(env, vc, n), heads, n_cts, n_cts, env.ctx.empty_ext(n))
        got = env.host(env.ctx.decode_context_hoisted(_tiled(env, a, n), None, heads, n_cts, d2, 1, rlk, list(keys), vext=ext,
                                                      sum_before_scaling=True))
        want = {}
        for h in range(heads):
            us = range(h * n_cts, (h + 1) * n_cts)
            first = us[0] % 6
            if first not in want:
                want[first] = attention.decode_context_hoisted(env.orc, [a[u % 3] for u in us], [vc[u % 2] for u in us], raw_rlk,
                                                               dict(zip(gs, raws)), d2, 1, sum_first=True)
            assert np.array_equal(got[h], want[first]), (name, heads, n_cts, h)
