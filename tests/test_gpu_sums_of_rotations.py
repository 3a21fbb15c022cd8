"""Summed rotations whose products are added up unreduced, eight between two reductions: one to 17 rotations, by rows (one unit to a workgroup), by
whole units, by pairs of units with the division by P, and from digits in memory, whose words are asked for a rotation ahead (odd and even
numbers), with the largest and the middle residues in ciphertexts and keys; bit-compared with the oracle.  Units repeat two distinct ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads import PRESETS
from workloads.params import ParamSet

from .bruteforce import ntt_primes
from .test_gpu_parity import Env, say

_P = ntt_primes(1 << 50, 2 << 13, 5)
SETS = {**PRESETS, "k4": ParamSet("n8192_k4_sums", 13, q=tuple(_P[:4]), p=tuple(_P[4:]), alpha=1)}
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


# 256 compute units, N = 8192: 48 units take 192 workgroups of one (unit, prime) each, 256 units one workgroup each (up to five rotations: keys of a
# prime fit an L2); N = 4096: 100 units 300 workgroups, 470 units one each.  1, 2 and 6 units: sums from digits in memory, one ciphertext to a thread, 12: two,
# both without words asked for ahead as well (one rotation, and more than nine).
# 460, 901 and 511 (a last pair of one): two units to a workgroup with the division by P, whole rounds of them and not
@pytest.mark.parametrize("name,batch,counts", [("C2", 48, (1, 2, 7, 8, 9, 16, 17)), ("C2", 256, (1, 2, 5)), ("C1", 100, (7, 8, 9)), ("C1", 470, (1, 8, 9)),
                                               ("C2", 1, (1, 2, 3, 6, 9)), ("C2", 12, (2, 5)), ("C5", 2, (2, 3)),
                                               ("C2", 6, (4, 11, 15)), ("C2", 12, (1, 15)),
                                               ("C2", 460, (7, 9)), ("C2", 901, (1, 8)), ("k4", 511, (3, 7))])
def test_numbers_of_rotations(name, batch, counts):
    env = _env(name)
    q = np.array(env.prm.q, dtype=np.uint64)[:, None]
    x = env.cts(61, 2)
    x[1, 0], x[1, 1] = q - 1, q // 2
    raws = [env.key(70)[0], np.empty_like(env.key(70)[0])]
    for r, p in enumerate(env.qp):
        raws[1][:, 0, r], raws[1][:, 1, r, ::2], raws[1][:, 1, r, 1::2] = p - 1, p // 2, p // 2 + 1
    keys = [env.ctx.ksk_prepare(env.dev(raw)) for raw in raws]
    xd = env.dev(np.ascontiguousarray(x[np.arange(batch) % 2]))
    for n in counts:
        say(f"{n} summed rotations {name}, {batch} units")
        gs = [2 * env.n - 1] + [pow(3, 1 + i, 2 * env.n) for i in range(n - 1)]
        want = [env.orc.rotate_sum_hoisted(x[b], gs, {g: raws[i % 2] for i, g in enumerate(gs)}) for b in range(2)]
        got = env.host(env.ctx.rotate_sum_hoisted(xd, gs, [keys[i % 2] for i in range(n)], batch))
        for b in range(batch):
            assert np.array_equal(got[b], want[b % 2]), (name, batch, n, b)
