"""Parameter sets cg_create accepts beside the presets, bit-compared with the oracle: more than three digits
(their products need a reduction that three do not), two special primes and digits of two primes at the smaller ring
degrees, one special prime at the largest.  Batches lie on both sides of every rule of the dispatch that
the set can reach; units repeat three distinct operands, so that every unit is checked."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads.params import ParamSet

from .bruteforce import ntt_primes
from .test_gpu_parity import Env, _block_keys, say


def _set(name, log2n, k, nsp, alpha):
    p = ntt_primes(1 << 50, 2 << log2n, k + nsp)
    return ParamSet(name, log2n, q=tuple(p[:k]), p=tuple(p[k:]), alpha=alpha)


SETS = {s.name: s for s in (_set("n8192_k4", 13, 4, 1, 1), _set("n4096_k5_2sp", 12, 5, 2, 1),
                            _set("n4096_k6", 12, 6, 1, 1), _set("n8192_k4_a2", 13, 4, 2, 2),
                            _set("n4096_k2_a2", 12, 2, 2, 2), _set("n8192_k6_2sp", 13, 6, 2, 1),
                            _set("n16384_k3", 14, 3, 1, 1))}
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


def _operands(env, seed):
    """three ciphertexts: random with extreme residues, all residues the largest, every second one zero"""
    x = env.cts(seed, 3)
    Q = int(np.prod([int(p) for p in env.prm.q], dtype=object))
    for i, m in enumerate(env.prm.q):
        x[0, :, i, :6] = [0, m - 1, (Q // 2) % m, (Q // 2 + 1) % m, (m - 1) // 2, (m + 1) // 2]
        x[1, :, i, :] = m - 1
    x[2, ..., ::2] = 0
    return x


def _tiled(env, x, batch):
    return env.dev(np.ascontiguousarray(x[np.arange(batch) % len(x)]))


def _check(env, got, want, what):
    for u, g in enumerate(env.host(got)):
        assert np.array_equal(g, want[u % 3]), (env.name, what, u)


@pytest.mark.parametrize("name,batches", [("n8192_k4", (1, 14, 15, 60)), ("n4096_k5_2sp", (2, 23, 24)),
                                          ("n4096_k6", (1, 20, 70)), ("n8192_k4_a2", (2, 40)),
                                          ("n4096_k2_a2", (3, 26, 120)), ("n8192_k6_2sp", (1, 10)),
                                          ("n16384_k3", (1, 18, 19, 40))])
def test_products(name, batches):
    env = _env(name)
    a, b = _operands(env, 10), env.cts(11, 3)
    b[1] = a[1]
    want = [env.orc.mul(a[i], b[i]) for i in range(3)]
    for batch in batches:
        say(f"mul {name} batch {batch}")
        _check(env, env.ctx.mul(_tiled(env, a, batch), _tiled(env, b, batch), batch), want, ("mul", batch))
    total = env.orc.mul_sum([a[i] for i in (0, 1, 2, 0, 1)], [b[i] for i in (0, 1, 2, 0, 1)])
    say(f"mul_sum {name}")
    got = env.host(env.ctx.mul_sum(_tiled(env, a, 5), _tiled(env, b, 5), 1, 5))
    assert np.array_equal(got[0], total), (name, "mul_sum")


# key switches of N / batch against 256 compute units: half a round of (unit, prime) rows, whole rounds, and whole units
@pytest.mark.parametrize("name,batches", [("n8192_k4", (1, 25, 26, 36, 60, 232)), ("n4096_k5_2sp", (1, 18, 30, 80)),
                                          ("n4096_k6", (1, 18, 19, 26, 60, 462)), ("n8192_k4_a2", (1, 40, 90)),
                                          ("n4096_k2_a2", (1, 70)), ("n8192_k6_2sp", (1, 17, 30)),
                                          ("n16384_k3", (1, 70))])
def test_key_switches(name, batches):
    env = _env(name)
    n, k = env.n, env.k
    x = _operands(env, 20)
    y = env.cts(21, 3)
    d = np.concatenate([x, y[:, :1]], axis=1)
    d[1, 2] = x[1, 0]
    raw, key = env.key(22)
    gs = [2 * n - 1, 3, 2 * n - 3, 9]
    raws, keys = zip(*[env.key(23 + i) for i in range(len(gs))])
    want = {"relin": [env.orc.relin(v, raw) for v in d], "rotate": [env.orc.rotate(v, 5, raw) for v in x],
            "sum": [env.orc.rotate_sum_hoisted(v, gs, dict(zip(gs, raws))) for v in x]}
    q = np.array(env.prm.q, dtype=np.uint64)[None, :, None]
    want["add"] = [(a + v) % q for a, v in zip(want["rotate"], x)]
    series = [[env.orc.rotate_hoisted(v, g, r) for v in x] for g, r in zip(gs, raws)]
    for batch in batches:
        say(f"key switches {name} batch {batch}")
        xd = _tiled(env, x, batch)
        _check(env, env.ctx.relin(_tiled(env, d, batch), key, batch), want["relin"], ("relin", batch))
        _check(env, env.ctx.rotate(xd, 5, key, batch), want["rotate"], ("rotate", batch))
        _check(env, env.ctx.rotate(xd, 5, key, batch, accumulate=True), want["add"], ("add", batch))
        _check(env, env.ctx.rotate_sum_hoisted(xd, gs, keys, batch), want["sum"], ("sum", batch))
        if batch <= 100:
            got = env.ctx.rotate_hoisted(xd, gs, keys, batch)
            for i in range(len(gs)):
                _check(env, got[:, i].contiguous(), series[i], ("hoisted", batch, i))


# pairs of units from 5/4 x 256 rows on with four digits and more (64 and 65 ciphertexts of five rows, 40 and 41 of eight; in
# launches of single transforms just below), and two rounds of pairs, the last unit alone (155)
@pytest.mark.parametrize("name,batches", [("n8192_k4", (63, 64, 65, 155)), ("n8192_k6_2sp", (39, 40, 41))])
def test_summed_rotations_of_pairs_of_units(name, batches):
    env = _env(name)
    x = _operands(env, 20)
    gs = [2 * env.n - 1, 3, 2 * env.n - 3, 9, 27, 2 * env.n - 9, 81, 5, 25]
    raws, keys = zip(*[env.key(23 + i) for i in range(len(gs))])
    for n_rot in (1, 9):
        want = [env.orc.rotate_sum_hoisted(v, gs[:n_rot], dict(zip(gs, raws))) for v in x]
        for batch in batches:
            say(f"{n_rot} rotations summed {name} batch {batch}")
            _check(env, env.ctx.rotate_sum_hoisted(_tiled(env, x, batch), gs[:n_rot], keys[:n_rot], batch), want, (n_rot, batch))


@pytest.mark.parametrize("name,batches", [("n4096_k6", (1, 40)), ("n8192_k6_2sp", (1,))])
def test_the_longest_sum_of_the_largest_values(name, batches):
    """128 rotations of six digits, every transformed digit and key value as large as it gets: constants are their own
    transforms and keep their value under every rotation.  (The integer accumulators hold 768 such products.)"""
    env = _env(name)
    n, n_rot = env.n, 128
    x = np.zeros((1, 2, env.k, n), dtype=np.uint64)
    x[0, :, :, 0] = [m - 1 for m in env.prm.q]
    raw = np.zeros((env.prm.dnum, 2, len(env.qp), n), dtype=np.uint64)
    raw[..., 0] = [(m - 1) // 2 for m in env.qp]
    key = env.ctx.ksk_prepare(env.dev(raw))
    gs = [pow(3, i, 2 * n) for i in range(1, n_rot + 1)]
    want = env.orc.rotate_sum_hoisted(x[0], gs, {g: raw for g in gs})
    for batch in batches:
        say(f"128 rotations summed {name} batch {batch}")
        got = env.host(env.ctx.rotate_sum_hoisted(_tiled(env, x, batch), gs, [key] * n_rot, batch))
        for u in range(batch):
            assert np.array_equal(got[u], want), (name, batch, u)


@pytest.mark.parametrize("name", ["n4096_k6", "n8192_k4_a2", "n16384_k3"])
def test_plain_products_and_appends(name):
    env = _env(name)
    n = env.n
    x = _operands(env, 30)
    rng = np.random.default_rng(31)
    pt = rng.integers(0, env.prm.t, (2, n), dtype=np.uint64)
    masks = env.ctx.plain_prepare(env.dev(pt))
    say(f"mul_plain and kv_append {name}")
    want = [env.orc.mul_plain(v, pt[0]) for v in x]
    _check(env, env.ctx.mul_plain(env.dev(x), masks, 3), want, "mul_plain")
    cache = env.dev(env.cts(32, 3))
    before = env.host(cache.clone())
    q = np.array(env.prm.q, dtype=np.uint64)[None, :, None]
    for tau in (0, 1):
        env.ctx.kv_append(cache, 1, 3, tau, env.dev(x), masks, n // 2)
        before = [(env.orc.mul_plain(v, pt[tau]) + (old if tau else 0)) % q for v, old in zip(x, before)]
        _check(env, cache.view(3, 2, env.k, n), before, ("kv_append", tau))


# rows of all caches: one to a workgroup, and several (512 workgroups of N = 8192 fill the chip, 256 of N = 16384)
@pytest.mark.parametrize("name,batches", [("n4096_k2_a2", (1, 300)), ("n8192_k4_a2", (1, 80)), ("n16384_k3", (2, 50))])
def test_appends_to_many_caches(name, batches):
    env = _env(name)
    x, old = _operands(env, 40), _operands(env, 41)
    pt = np.random.default_rng(42).integers(0, env.prm.t, (2, env.n), dtype=np.uint64)
    masks = env.ctx.plain_prepare(env.dev(pt))
    q = np.array(env.prm.q, dtype=np.uint64)[None, :, None]
    first = [env.orc.mul_plain(v, pt[0]) for v in x]
    more = [(env.orc.mul_plain(v, pt[1]) + w) % q for v, w in zip(x, old)]
    for batch in batches:
        say(f"kv_append {name}: {batch} caches")
        cache, rows = _tiled(env, old, batch), _tiled(env, x, batch)
        env.ctx.kv_append(cache, 1, batch, 1, rows, masks, env.n // 2)
        _check(env, cache, more, ("added", batch))
        env.ctx.kv_append(cache, 1, batch, 0, rows, masks, env.n // 2)
        _check(env, cache, first, ("fresh", batch))


# sums over one copy of the token, and many; rows of all matrices: below a workgroup each, and several
@pytest.mark.parametrize("name,n_diag,units", [("n4096_k6", 1, 2), ("n4096_k2_a2", 16, 300), ("n8192_k4_a2", 32, 3),
                                               ("n8192_k4", 2, 80), ("n16384_k3", 1, 50), ("n16384_k3", 8, 2)])
def test_vector_matrix_products(name, n_diag, units):
    from oracle import attention
    env = _env(name)
    n, d2 = env.n, env.n // 4
    x = _operands(env, 50)[1]
    pt = np.random.default_rng(51).integers(0, env.prm.t, (2, n_diag, n), dtype=np.uint64)
    pt[0, :, ::2] = env.prm.t - 1
    shift = [pow(3, sh, 2 * n) for sh in attention.cpvm_shifts(n_diag)]
    block = _block_keys(env, d2)
    keys = {g: env.key(60 + i) for i, g in enumerate(sorted(set(shift + block)))}
    raw = {g: keys[g][0] for g in keys}
    say(f"cpvm {name}: {units} matrices of {n_diag} diagonals")
    diags = env.ctx.plain_prepare(env.dev(np.ascontiguousarray(pt[np.arange(units) % 2].reshape(-1, n))))
    got = env.host(env.ctx.cpvm(env.dev(x[None]), diags, units, n_diag, d2, [keys[g][1] for g in shift],
                                [keys[g][1] for g in block]))
    want = [attention.cpvm(env.orc, x, list(pt[i]), raw, d2) for i in range(2)]
    for u in range(units):
        assert np.array_equal(got[u], want[u % 2]), (name, u)


# rows for one round and a half of workgroups (from there on waves have priorities), and a row less: 4, 2 and 1 workgroups to
# each of 256 compute units, forward; inverse N = 8192 has one
@pytest.mark.parametrize("name,rows", [("n4096_k6", (1535, 1536)), ("n8192_k4", (383, 384, 767, 768)), ("n16384_k3", (383, 384))])
def test_transforms_of_many_rows(name, rows):
    env = _env(name)
    primes = len(env.qp)
    base = np.stack([np.random.default_rng(70 + i).integers(0, m, env.n, dtype=np.uint64) for i, m in enumerate(env.qp)])
    base[:, 0] = 0
    base[:, 1::2] = np.array(env.qp, dtype=np.uint64)[:, None] - 1
    from oracle import bfv
    want = np.stack([bfv.ntt_forward(base[i], m) for i, m in enumerate(env.qp)])
    for n in rows:
        say(f"ntt {name}: {n} rows")
        idx = [i % primes for i in range(n)]
        x = env.dev(base[idx])
        got = env.ctx.ntt_forward(x, idx)
        assert np.array_equal(env.host(got), want[idx]), (name, n)
        assert np.array_equal(env.host(env.ctx.ntt_inverse(got, idx)), base[idx]), (name, n)
