"""Series of rotations of the same ciphertexts in one launch behind the mod-up (rot_row_kernel): one to three digits, whose values come in block by block
and are permuted in LDS, Galois elements that leave the blocks where they are and such as move them furthest, more workgroups than compute
units and a ragged last round, the largest residues in ciphertexts and keys; bit-compared with the oracle.  Units repeat two distinct ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from workloads import PRESETS
from workloads.params import ParamSet

from .bruteforce import ntt_primes
from .test_gpu_parity import Env, say


def _set(log2n, k):
    p = ntt_primes(1 << 50, 2 << log2n, k + 1)
    return ParamSet(f"n{1 << log2n}_k{k}_rows", log2n, q=tuple(p[:k]), p=tuple(p[k:]), alpha=1)


# 2 x rotations x ciphertexts workgroups, from half as many as the 256 compute units on
@pytest.mark.parametrize("prm,batch,count", [(PRESETS["C2"], 3, 66), (_set(13, 2), 5, 29), (_set(13, 1), 9, 15), (PRESETS["C1"], 3, 130), (_set(12, 3), 13, 11)],
                         ids=lambda v: getattr(v, "name", str(v)))
def test_series(prm, batch, count):
    import paper_2602_08798_amd as P
    from oracle import Oracle
    env = Env.__new__(Env)
    env.P, env.name, env.prm, env.ctx, env.orc = P, prm.name, prm, P.Context(prm), Oracle(prm)
    env.n, env.k, env.qp, env._keys = prm.n, prm.k, list(prm.q) + list(prm.p), {}
    n = env.n
    x = env.cts(81, 2)
    x[1, 0], x[1, 1] = (np.array(prm.q, dtype=np.uint64)[:, None] - 1 for _ in range(2))
    raws = [env.key(90)[0], np.empty_like(env.key(90)[0])]
    for r, p in enumerate(env.qp):
        raws[1][:, 0, r], raws[1][:, 1, r, ::2], raws[1][:, 1, r, 1::2] = p - 1, p // 2, p // 2 + 1
    keys = [env.ctx.ksk_prepare(env.dev(raw)) for raw in raws]
    # 2N - 1 and N + 1 change the highest bits of an exponent, n / 64 + 1 leaves the lowest six; powers of 3 in between
    gs = ([2 * n - 1, n + 1, n // 64 + 1, 3] + [pow(3, 5 * i + 2, 2 * n) for i in range(count)])[:count]
    say(f"{count} hoisted rotations {prm.name}, {batch} units")
    got = env.host(env.ctx.rotate_hoisted(env.dev(np.ascontiguousarray(x[np.arange(batch) % 2])), gs, [keys[i % 2] for i in range(count)], batch))
    for u in range(2):
        want = env.orc.rotate_many(x[u], gs, {g: raws[i % 2] for i, g in enumerate(gs)})
        for b in range(u, batch, 2):
            for i in range(count):
                assert np.array_equal(got[b, i], want[i]), (prm.name, b, i)
    env.ctx.close()
