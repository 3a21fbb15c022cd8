"""No kernel is compiled that no call launches.  Runs without a GPU, against a recording stand-in for the runtime: every ring
degree, number and kind of primes that a context takes, with batches on both sides of the dispatch's limits."""
import json
import sys

import pytest

from tests.bruteforce import ntt_primes
from tests.stubbed import DEV as d, Stubbed, run, u32, vp
from workloads.params import ParamSet

SHAPES = [(k, nsp, alpha) for k in range(1, 7) for nsp, alpha in ((1, 1), (2, 1), (2, 2)) if k % alpha == 0 and (k, nsp) != (3, 2)]
BATCHES = (1, 2, 4, 10, 13, 20, 43, 60, 64, 107, 200, 256, 512, 800)


def _unreached(lib):
    seen = set()
    gs, keys, out = (u32 * 64)(*range(3, 131, 2)), (vp * 5000)(*[1 << 20] * 5000), vp(1 << 40)
    f = lib.lib
    for log2n in (12, 13, 14):
        for k, nsp, alpha in SHAPES:
            p = ntt_primes(1 << 50, 2 << log2n, k + nsp)
            ctx = lib.create(ParamSet("x", log2n, q=tuple(p[:k]), p=tuple(p[k:]), alpha=alpha))

            def go(name, *args):
                seen.update(x[0] for x in lib.kernels(lambda: getattr(f, name)(ctx, None, *args)))

            for batch in BATCHES:
                b, rows = u32(batch), (u32 * batch)(*[i % k for i in range(batch)])
                go("cg_mul", d, d, out, b, u32(1), d)
                go("cg_mul", d, d, out, b, u32(3), d)
                go("cg_mul_sum", d, d, out, b, u32(2), d)
                go("cg_mul_sum", d, d, out, b, u32(7), d)
                go("cg_relin", d, d, out, b, d)
                go("cg_rotate", d, u32(3), d, out, b, 1, d)
                go("cg_rotate_sum_hoisted", d, u32(1), gs, keys, out, b, d)
                go("cg_rotate_sum_hoisted", d, u32(7), gs, keys, out, b, d)
                go("cg_rotate_hoisted", d, u32(4), gs, keys, out, b, d)
                go("cg_mul_plain", d, d, u32(0), out, b, d)
                go("cg_plain_prepare", d, out, b)
                go("cg_kv_append", d, u32(2), b, u32(1), d, d, u32(64), d)
                go("cg_cache_extend", d, b, u32(1), u32(1), out)
                go("cg_ntt_forward", d, out, rows, b)
                go("cg_ntt_inverse", d, out, rows, b)
                go("cg_add", d, d, out, u32(2), b)
                go("cg_add_plain", d, d, u32(1), 0, out, b)
                if batch <= 64:
                    for ext in (None, d):
                        for cts in (1, 2, 5):
                            go("cg_decode_scores_hoisted", d, d, ext, b, u32(cts), u32(cts), u32(64), u32(3), d, keys, out, d)
                            for sums in (0, 1):
                                go("cg_decode_context_hoisted", d, d, ext, b, u32(cts), u32(cts), u32(64), u32(3), sums, d, keys,
                                   out, d)
                    for n_diag in (8, 64):
                        go("cg_cpvm", d, d, b, u32(n_diag), u32(64), keys, keys, out, d)
                        go("cg_cpvm_hoisted", d, d, b, u32(n_diag), u32(64), u32(3), keys, keys, out, d)
                    go("cg_decode_scores_outer", d, d, b, u32(16), d, d, keys, out, d)
                if batch <= 10:
                    go("cg_prefill_av_hoisted", d, d, b, u32(64), 1, d, keys, out, d)
                    go("cg_prefill_repack", d, b, u32(64), d, keys, out, d)
            go("cg_decode_scores_outer", d, d, u32(260), u32(16), d, d, keys, out, d)
            go("cg_ksk_prepare", d, out)
            assert f.cg_destroy(ctx) == 0
    return sorted(set(lib.compiled()) - seen)


@pytest.fixture(scope="module")
def unreached(tmp_path_factory):
    return run(__file__, tmp_path_factory.mktemp("stub"))


# a key has up to 96 rows: more than the compute units of a partition of the chip, never of 256
ELSEWHERE = ("bench_exchange_kernel", "bench_modmul_kernel", "ntt_fwd_kernel<13, 16, LdRowsU64, StF64Red>")


def test_every_kernel_is_reached(unreached):
    assert [k for k in unreached if k not in ELSEWHERE] == []


if __name__ == "__main__":
    print(json.dumps(_unreached(Stubbed(*sys.argv[1:]))))
