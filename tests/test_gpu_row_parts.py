"""Launches of few rows take every row in two or four parts: transforms, relinearisations and summed rotations (and rotations, whose rows stay whole) on both sides of the
row counts where the number of parts changes (256 compute units), bit-compared with the oracle.  Rows and units repeat
a few distinct ones; the largest residues are among them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads import PRESETS
from workloads.params import ParamSet

from .bruteforce import ntt_primes
from .test_gpu_parity import Env, say

SETS = {"C1": PRESETS["C1"], "C2": PRESETS["C2"], "C5": PRESETS["C5"],
        # digits of two primes, and one digit (the sums' rows stay where they are), at N = 8192
        "pairs": ParamSet("n8192_k2_a2", 13, q=tuple(ntt_primes(1 << 50, 2 << 13, 2)),
                          p=tuple(ntt_primes(1 << 49, 2 << 13, 2)), alpha=2),
        "one": ParamSet("n8192_k1", 13, q=tuple(ntt_primes(1 << 50, 2 << 13, 1)),
                        p=tuple(ntt_primes(1 << 49, 2 << 13, 1)), alpha=1)}
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


@pytest.mark.parametrize("name", ["C1", "C2", "C5"])
def test_transforms_of_few_rows(name):
    from oracle import bfv
    env = _env(name)
    L = env.k + env.prm.nsp
    rng = np.random.default_rng(7)
    few = np.stack([rng.integers(0, p, env.n, dtype=np.uint64) for p in env.qp])
    few[0, :], few[1, ::2] = env.qp[0] - 1, env.qp[1] - 1
    fwd = [bfv.ntt_forward(few[i], int(env.qp[i])) for i in range(L)]
    inv = [bfv.ntt_inverse(few[i], int(env.qp[i])) for i in range(L)]
    for rows in (1, 3, 63, 64, 65, 85, 86, 128, 129) + ((257, 352, 353) if name == "C2" else ()):
        say(f"transforms {name}, {rows} rows")
        idx = [i % L for i in range(rows)]
        x = env.dev(np.ascontiguousarray(few[idx]))
        f, g = env.host(env.ctx.ntt_forward(x, idx)), env.host(env.ctx.ntt_inverse(x, idx))
        for i in range(rows):
            assert np.array_equal(f[i], fwd[i % L]), (name, rows, i)
            assert np.array_equal(g[i], inv[i % L]), (name, rows, i)


# rows of the mod-up, then of the inverse transforms, per unit: C1 6 and 6, C2 12 and 8, C5 24 and 16, pairs 4 and 8, one 2 and 4
@pytest.mark.parametrize("name,batches", [("C1", (1, 10, 11, 21, 22)), ("C2", (1, 4, 5, 6, 10, 11, 33, 40)), ("C5", (1, 2, 3, 4, 5)),
                                          ("pairs", (2, 10, 11, 16, 17)), ("one", (1, 21, 22, 32, 33))])
def test_key_switches_of_few_units(name, batches):
    env = _env(name)
    x = env.cts(21, 2)
    x[1, 1] = np.array(env.prm.q, dtype=np.uint64)[:, None] - 1
    gs = [3, 2 * env.n - 1, pow(3, 5, 2 * env.n)]
    keys = [env.key(30 + i) for i in range(3)]
    d3 = np.concatenate([x, x[::-1, 1:]], axis=1)
    rot = [env.orc.rotate(x[b], gs[0], keys[0][0]) for b in range(2)]
    relin = [env.orc.relin(d3[b], keys[1][0]) for b in range(2)]
    sums = [env.orc.rotate_sum_hoisted(x[b], gs, {g: k[0] for g, k in zip(gs, keys)}) for b in range(2)]
    for batch in batches:
        say(f"key switches {name}, {batch} units")
        xd = env.dev(np.ascontiguousarray(x[np.arange(batch) % 2]))
        got = env.host(env.ctx.rotate(xd, gs[0], keys[0][1], batch))
        got_relin = env.host(env.ctx.relin(env.dev(np.ascontiguousarray(d3[np.arange(batch) % 2])), keys[1][1], batch))
        got_sum = env.host(env.ctx.rotate_sum_hoisted(xd, gs, [k[1] for k in keys], batch))
        for b in range(batch):
            assert np.array_equal(got[b], rot[b % 2]), (name, batch, b)
            assert np.array_equal(got_relin[b], relin[b % 2]), (name, batch, b)
            assert np.array_equal(got_sum[b], sums[b % 2]), (name, batch, b)
