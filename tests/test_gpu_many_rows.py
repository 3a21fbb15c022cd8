"""Inverse transforms of callers' rows on both sides of the row count from which a row runs on 512 threads (N = 8192: three rows to two of
the 256 compute units), several rounds of workgroups with a ragged last one, into another buffer and in place; bit-compared
with the oracle.  Rows repeat a few distinct ones; the largest residues are among them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from .test_gpu_parity import say
from .test_gpu_row_parts import _env


@pytest.mark.parametrize("name,rows", [("C2", (384, 385, 513, 1100)), ("C5", (257, 600))])
def test_inverse_transforms(name, rows):
    from oracle import bfv
    env = _env(name)
    L = env.k + env.prm.nsp
    rng = np.random.default_rng(9)
    few = np.stack([rng.integers(0, p, env.n, dtype=np.uint64) for p in env.qp])
    few[0, :], few[1, ::2], few[2, 1::2] = env.qp[0] - 1, env.qp[1] - 1, env.qp[2] // 2
    want = env.dev(np.stack([bfv.ntt_inverse(few[i], int(env.qp[i])) for i in range(L)]))
    for n in rows:
        say(f"inverse transforms {name}, {n} rows")
        idx = [i % L for i in range(n)]
        x = env.dev(few)[idx].contiguous()
        got = env.ctx.ntt_inverse(x, idx)
        assert bool((got == want[idx]).all()), (name, n)
        env.ctx.ntt_inverse(x, idx, out=x)
        assert bool((x == want[idx]).all()), (name, n, "in place")
