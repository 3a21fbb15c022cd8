"""The kernels that take one (unit, prime) through several transforms in a workgroup, at the batches where
the dispatch changes (a product has 2k + 1 rows, a key switch k + nsp, against 256 compute units) and over several rounds
of workgroups: bit-compared with the oracle.  Units repeat a few distinct operands, so that every unit of
a large batch is checked.  Parameter sets: the benchmark's, the smallest ones, and primes of different
sizes (the lazily reduced values are bounded by the largest prime's size, not by the row's own prime)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads import PRESETS
from workloads.params import ParamSet

from .bruteforce import ntt_primes
from .test_gpu_parity import Env, say

MIXED = ParamSet("mixed_n8192_k3", 13,
                 q=tuple(p for b in (50, 43, 48) for p in ntt_primes(1 << b, 2 << 13, 1)),
                 p=tuple(ntt_primes((1 << 50) - (1 << 45), 2 << 13, 1)), alpha=1)
SETS = {"C1": PRESETS["C1"], "C2": PRESETS["C2"], "mixed": MIXED,
        "k1": ParamSet("n8192_k1", 13, q=tuple(ntt_primes(1 << 50, 2 << 13, 1)),
                       p=tuple(ntt_primes(1 << 49, 2 << 13, 1)), alpha=1),
        "k3": ParamSet("n4096_k3", 12, q=tuple(ntt_primes(1 << 50, 2 << 12, 3)),
                       p=tuple(ntt_primes(1 << 49, 2 << 12, 1)), alpha=1)}
_envs = {}


def _env(name):
    if name not in _envs:
        env = Env.__new__(Env)
        import paper_2602_08798_amd as P
        from oracle import Oracle
        prm = SETS[name]
        env.P, env.name, env.prm, env.ctx, env.orc = P, name, prm, P.Context(prm), Oracle(prm)
        env.n, env.k, env.qp, env._keys = prm.n, prm.k, list(prm.q) + list(prm.p), {}
        _envs[name] = env
    return _envs[name]


def _extremes(env, x):
    """residues at the ends and around the middle of the range of the lift"""
    Q = int(np.prod([int(p) for p in env.prm.q], dtype=object))
    for i, m in enumerate(env.prm.q):
        x[0, 0, i, :6] = [0, m - 1, (Q // 2) % m, (Q // 2 + 1) % m, (m - 1) // 2, (m + 1) // 2]
        x[1, 1, i, :] = m - 1
    return x


def _tiled(env, x, batch):
    return env.dev(np.ascontiguousarray(x[np.arange(batch) % len(x)]))


# rows of a batch: C2 and mixed 7 per product and 4 per key switch, C1 5 and 3, k1 3 and 2, k3 7 and 4
@pytest.mark.parametrize("name,batches", [("C2", (18, 19, 36, 37, 55, 63, 64, 74, 150)), ("C1", (25, 26, 43, 120)),
                                          ("mixed", (19, 74)), ("k1", (43, 260)), ("k3", (37, 80))])
def test_products_and_relinearisation_at_the_edges_of_the_dispatch(name, batches):
    env = _env(name)
    raw, rlk = env.key(20)
    a, b = _extremes(env, env.cts(10, 3)), _extremes(env, env.cts(11, 2))
    want = {(i, j): env.orc.mul(a[i], b[j]) for i in range(3) for j in range(2)}
    relin = {key: env.orc.relin(w, raw) for key, w in want.items()}
    for batch in batches:
        say(f"mul and mul_relin {name} batch {batch}")
        ad, bd = _tiled(env, a, batch), _tiled(env, b, batch)
        got3 = env.host(env.ctx.mul(ad, bd, batch))
        got2 = env.host(env.ctx.mul_relin(ad, bd, rlk, batch))
        for u in range(batch):
            assert np.array_equal(got3[u], want[u % 3, u % 2]), (name, batch, u)
            assert np.array_equal(got2[u], relin[u % 3, u % 2]), (name, batch, u)


@pytest.mark.parametrize("name,batch,group", [("C2", 66, 3), ("C2", 64, 64), ("C1", 60, 4), ("mixed", 20, 2)])
def test_products_with_a_shared_operand(name, batch, group):
    env = _env(name)
    a, b = _extremes(env, env.cts(12, -(-batch // group))) if batch // group > 1 else env.cts(12, 1), env.cts(13, 2)
    say(f"mul {name} batch {batch}, one a operand for {group}")
    got = env.host(env.ctx.mul(env.dev(a), _tiled(env, b, batch), batch, a_group=group))
    for u in range(batch):
        assert np.array_equal(got[u], env.orc.mul(a[u // group], b[u % 2])), (name, batch, u)


@pytest.mark.parametrize("name,shapes", [("C2", ((1, 32), (3, 7), (1, 75))), ("C1", ((4, 16), (12, 4))),
                                         ("mixed", ((1, 20),)), ("k1", ((5, 9),)), ("k3", ((2, 11),))])
def test_sums_of_products_in_parts(name, shapes):
    """long groups cut into even and uneven parts, the largest residues in every third unit"""
    env = _env(name)
    a, b = _extremes(env, env.cts(14, 3)), _extremes(env, env.cts(15, 2))
    a[1], b[1] = [[[m - 1] * env.n for m in env.prm.q]] * 2, [[[m - 1] * env.n for m in env.prm.q]] * 2
    for groups, group in shapes:
        say(f"mul_sum {name}: {groups} groups of {group}")
        units = np.arange(groups * group)
        got = env.host(env.ctx.mul_sum(_tiled(env, a, len(units)), _tiled(env, b, len(units)), groups, group))
        for g in range(groups):
            us = units[g * group:(g + 1) * group]
            assert np.array_equal(got[g], env.orc.mul_sum([a[u % 3] for u in us], [b[u % 2] for u in us])), (name, groups, group, g)


@pytest.mark.parametrize("name,shapes", [("C2", ((13, 8), (16, 9), (5, 36), (8, 25))), ("mixed", ((13, 8), (3, 60))),
                                         ("k1", ((34, 7), (3, 86)))])
def test_sums_of_products_in_ranges_across_groups(name, shapes):
    """units of all groups in equal ranges: groups inside one range, ends of groups and of ranges together and apart"""
    env = _env(name)
    a, b = _extremes(env, env.cts(16, 3)), _extremes(env, env.cts(17, 2))
    for groups, group in shapes:
        say(f"mul_sum {name}: {groups} groups of {group}")
        units = np.arange(groups * group)
        got = env.host(env.ctx.mul_sum(_tiled(env, a, len(units)), _tiled(env, b, len(units)), groups, group))
        want = {}
        for g in range(groups):
            us = units[g * group:(g + 1) * group]
            key = us[0] % 6                                     # (the operands repeat every six units)
            if key not in want:
                want[key] = env.orc.mul_sum([a[u % 3] for u in us], [b[u % 2] for u in us])
            assert np.array_equal(got[g], want[key]), (name, groups, group, g)


@pytest.mark.parametrize("name,batches", [("C2", (31, 32, 65, 96, 130)), ("C1", (42, 43, 100)), ("mixed", (33,))])
def test_rotations_at_the_edges_of_the_dispatch(name, batches):
    env = _env(name)
    raw, gk = env.key(30)
    x = _extremes(env, env.cts(31, 3))
    x[2, :, :, :3] = 0
    for g in (3, 2 * env.n - 1):
        want = [env.orc.rotate(x[i], g, raw) for i in range(3)]
        for batch in batches:
            say(f"rotate {name} g={g} batch {batch}")
            got = env.host(env.ctx.rotate(_tiled(env, x, batch), g, gk, batch))
            for u in range(batch):
                assert np.array_equal(got[u], want[u % 3]), (name, g, batch, u)


@pytest.mark.parametrize("name,batches,n_rot", [("C2", (38, 39, 64, 96, 103, 195), 3), ("C1", (42, 43, 90), 9),
                                                ("mixed", (39,), 2), ("C2", (48,), 17)])
def test_rotation_sums_at_the_edges_of_the_dispatch(name, batches, n_rot):
    """also more rotations than are summed between two reductions"""
    env = _env(name)
    n = env.n
    gs = ([2 * n - 1, 3, 1, 2 * n - 3] + [pow(3, 5 * i + 2, 2 * n) for i in range(n_rot)])[:n_rot]
    keys = [env.key(40 + i % 3) for i in range(n_rot)]
    x = _extremes(env, env.cts(41, 3))
    x[2, :, :, ::3] = 0
    want = [env.orc.rotate_sum_hoisted(x[i], gs, {g: keys[i][0] for i, g in enumerate(gs)}) for i in range(3)]
    for batch in batches:
        say(f"rotate_sum_hoisted {name} batch {batch}, {n_rot} rotations")
        got = env.host(env.ctx.rotate_sum_hoisted(_tiled(env, x, batch), gs, [k[1] for k in keys], batch))
        for u in range(batch):
            assert np.array_equal(got[u], want[u % 3]), (name, batch, u)


@pytest.mark.parametrize("name,shapes", [("C2", ((1, 63), (1, 64), (5, 13), (2, 127), (40, 7))), ("C1", ((9, 9), (3, 86))),
                                         ("mixed", ((3, 22),)), ("k1", ((66, 1), (1, 130)))])
def test_hoisted_series_at_the_edges_of_the_dispatch(name, shapes):
    """more rotations than one launch takes, an output stride longer than the series, the largest residues"""
    env = _env(name)
    n = env.n
    x = _extremes(env, env.cts(51, 3))
    x[2, :, :, ::3] = 0
    for batch, n_rot in shapes:
        gs = ([2 * n - 1, 3, 1, 2 * n - 3] + [pow(3, 5 * i + 2, 2 * n) for i in range(n_rot)])[:n_rot]
        keys = [env.key(40 + i % 3) for i in range(n_rot)]
        say(f"rotate_hoisted {name} batch {batch}, {n_rot} rotations")
        got = env.host(env.ctx.rotate_hoisted(_tiled(env, x, batch), gs, [k[1] for k in keys], batch))
        for i in range(n_rot):
            want = [env.orc.rotate_hoisted(x[j], gs[i], keys[i][0]) for j in range(min(batch, 3))]
            for u in range(batch):
                assert np.array_equal(got[u, i], want[u % 3]), (name, batch, n_rot, u, i)


# units against 256 compute units: whole key switches per workgroup from 231 (N = 8192) and 461 (N = 4096) on
@pytest.mark.parametrize("name,batches", [("C2", (230, 231, 480)), ("C1", (256, 460, 461, 700)), ("mixed", (256,)),
                                          ("k1", (250,)), ("k3", (512,))])
def test_key_switches_at_the_edges_of_the_dispatch(name, batches):
    env = _env(name)
    n, k = env.n, env.k
    x = _extremes(env, env.cts(61, 3))
    x[2, :, :, ::3] = 0
    y = env.cts(62, 2)
    d = np.stack([np.concatenate([x[i], y[i % 2, :1]]) for i in range(3)])
    raw, key = env.key(60)
    gs = [2 * n - 1, 3, 2 * n - 3, 9, 27][:5 if name == "C1" else 3]
    keys = [env.key(40 + i % 3) for i in range(len(gs))]
    g = 5
    want = {"relin": [env.orc.relin(v, raw) for v in d], "rotate": [env.orc.rotate(v, g, raw) for v in x],
            "sum": [env.orc.rotate_sum_hoisted(v, gs, {g: keys[i][0] for i, g in enumerate(gs)}) for v in x]}
    q = np.array(env.prm.q, dtype=np.uint64)[None, None, :, None]
    want["add"] = [(a + v) % q[0] for a, v in zip(want["rotate"], x)]
    for batch in batches:
        say(f"key switches {name} batch {batch}")
        xd = _tiled(env, x, batch)
        got = {"relin": env.ctx.relin(_tiled(env, d, batch), key, batch), "rotate": env.ctx.rotate(xd, g, key, batch),
               "add": env.ctx.rotate(xd, g, key, batch, accumulate=True),
               "sum": env.ctx.rotate_sum_hoisted(xd, gs, [v[1] for v in keys], batch)}
        for op, out in got.items():
            out = env.host(out)
            for u in range(batch):
                assert np.array_equal(out[u], want[op][u % 3]), (name, op, batch, u)


# both sides of the limits for idle units where a rotation's and a sum's differ from a relinearisation's
@pytest.mark.parametrize("name,batches", [("C2", (42, 43, 97, 140, 141)), ("C1", (43, 44, 123, 124)), ("k3", (42, 44, 83, 90))])
def test_rotations_and_sums_at_the_limits_for_idle_units(name, batches):
    env = _env(name)
    raw, gk = env.key(30)
    raw2, gk2 = env.key(31)
    x = _extremes(env, env.cts(33, 3))
    x[2, :, :, ::3] = 0
    gs = [2 * env.n - 1, 3]
    want = {"rotate": [env.orc.rotate(v, 9, raw) for v in x],
            "sum": [env.orc.rotate_sum_hoisted(v, gs, {gs[0]: raw, gs[1]: raw2}) for v in x]}
    for batch in batches:
        say(f"rotate and rotate_sum_hoisted {name} batch {batch}")
        xd = _tiled(env, x, batch)
        got = {"rotate": env.host(env.ctx.rotate(xd, 9, gk, batch)),
               "sum": env.host(env.ctx.rotate_sum_hoisted(xd, gs, [gk, gk2], batch))}
        for op, out in got.items():
            for u in range(batch):
                assert np.array_equal(out[u], want[op][u % 3]), (name, op, batch, u)


def test_scores_of_single_ciphertext_caches_with_a_transformed_copy():
    """one cache ciphertext per head: the query in coefficients times the transformed cache"""
    from oracle import attention
    env = _env("C2")
    heads, d2 = 20, 2
    raw_rlk, rlk = env.key(70)
    g = attention.fold_generators(env.n, d2)[0]
    raw_g, gk = env.key(71)
    q, kc = env.cts(72, 2), env.cts(73, 3)
    say(f"decode_scores_ext of {heads} heads, one ciphertext each")
    ext = env.ctx.empty_ext(heads)
    env.ctx.cache_extend(_tiled(env, kc, heads), heads, 1, 1, ext)
    got = env.host(env.ctx.decode_scores_ext(_tiled(env, q, heads), ext, heads, 1, d2, rlk, [gk]))
    for h in range(heads):
        want = attention.decode_scores(env.orc, q[h % 2], kc[h % 3], raw_rlk, {g: raw_g}, d2)
        assert np.array_equal(got[h, 0], want), h


@pytest.mark.parametrize("name,shapes", [("C1", ((1, 1), (3, 7), (85, 1), (43, 2))), ("k3", ((2, 5),))])
def test_context_sums_with_a_transformed_copy_in_parts(name, shapes):
    """N = 4096: products with a transformed cache summed in one launch (one part per group, several, several rounds), and just
    more of them than that is taken for"""
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


# three rows a product and prime in the transform that forms them: with no more rows than compute units, and just more
@pytest.mark.parametrize("name,batches", [("C2", (12, 13)), ("mixed", (1, 12)), ("k1", (28, 29))])
def test_products_of_few_rows(name, batches):
    env = _env(name)
    a, b = _extremes(env, env.cts(94, 3)), _extremes(env, env.cts(95, 2))
    want = {(i, j): env.orc.mul(a[i], b[j]) for i in range(3) for j in range(2)}
    for batch in batches:
        say(f"products {name} batch {batch}")
        got = env.host(env.ctx.mul(_tiled(env, a, batch), _tiled(env, b, batch), batch))
        for u in range(batch):
            assert np.array_equal(got[u], want[u % 3, u % 2]), (name, batch, u)


# pairs of units at N = 8192 (107 and 193, 128, 255 and 385: where whole rounds of pairs are few enough), and what is taken around
# them; an odd batch's last unit is alone; keys are read ahead over the end of a rotation, sums reduced after eight
@pytest.mark.parametrize("name,batches", [("C2", (79, 80, 107, 193, 385)), ("mixed", (81, 128)), ("k1", (160, 255, 385))])
def test_summed_rotations_of_pairs_of_units(name, batches):
    env = _env(name)
    n = env.n
    gs = [2 * n - 1, 3, 2 * n - 3, 9, 27, 2 * n - 9, 81, 5, 25]
    raws, keys = zip(*[env.key(100 + i) for i in range(len(gs))])
    x = _extremes(env, env.cts(96, 3))
    for n_rot in (1, 8, 9):
        want = [env.orc.rotate_sum_hoisted(v, gs[:n_rot], dict(zip(gs, raws))) for v in x]
        for batch in batches:
            say(f"{n_rot} rotations summed {name} batch {batch}")
            got = env.host(env.ctx.rotate_sum_hoisted(_tiled(env, x, batch), gs[:n_rot], keys[:n_rot], batch))
            for u in range(batch):
                assert np.array_equal(got[u], want[u % 3]), (name, n_rot, batch, u)
