"""Key switches at N = 16384 from digits to accumulators in one launch (ks_wide_kernel): relinearisations and summed rotations that read their
own half of a row, the other one, or both kinds, with digits of one and of two primes, several rounds of workgroups and a
ragged last one; bit-compared with the oracle.  Units repeat two distinct ones; the largest residues are among them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads import PRESETS
from workloads.params import ParamSet

from .bruteforce import ntt_primes
from .test_gpu_parity import Env, say

SETS = {"C5": PRESETS["C5"],
        "one_special": ParamSet("n16384_k2", 14, q=tuple(ntt_primes(1 << 50, 2 << 14, 2)),
                                p=tuple(ntt_primes(1 << 49, 2 << 14, 1)), alpha=1)}


# rows per unit: C5 8, one_special 3; one round of 256 compute units from 176 rows on, two from 368
@pytest.mark.parametrize("name,batches", [("C5", (21, 22, 32, 46, 80)), ("one_special", (58, 59, 85, 125))])
def test_summed_rotations_and_relinearisations(name, batches):
    import paper_2602_08798_amd as P
    from oracle import Oracle
    env, prm = Env.__new__(Env), SETS[name]
    env.P, env.name, env.prm, env.ctx, env.orc = P, name, prm, P.Context(prm), Oracle(prm)
    env.n, env.k, env.qp, env._keys = prm.n, prm.k, list(prm.q) + list(prm.p), {}
    n = env.n
    x, y = env.cts(41, 2), env.cts(42, 2, 3)
    x[1, 1] = y[1, 2] = np.array(prm.q, dtype=np.uint64)[:, None] - 1
    keys = [env.key(50 + i) for i in range(3)]
    # 3 and 2N - 1 exchange the halves, 3^2 does not; nine rotations have a reduction on the way
    series = ([2 * n - 1], [9, 3, 2 * n - 1], [pow(3, 1 + i, 2 * n) for i in range(9)])
    want = [[env.orc.rotate_sum_hoisted(x[b], gs, {g: keys[i % 3][0] for i, g in enumerate(gs)}) for b in range(2)] for gs in series]
    relin = [env.orc.relin(y[b], keys[0][0]) for b in range(2)]
    for batch in batches:
        say(f"wide key switches {name}, {batch} units")
        two = np.arange(batch) % 2
        xd, yd = env.dev(np.ascontiguousarray(x[two])), env.dev(np.ascontiguousarray(y[two]))
        for gs, w in zip(series, want):
            got = env.host(env.ctx.rotate_sum_hoisted(xd, gs, [keys[i % 3][1] for i in range(len(gs))], batch))
            for b in range(batch):
                assert np.array_equal(got[b], w[b % 2]), (name, batch, len(gs), b)
        got = env.host(env.ctx.relin(yd, keys[0][1], batch))
        for b in range(batch):
            assert np.array_equal(got[b], relin[b % 2]), (name, batch, b)
    env.ctx.close()
