"""Which kernel a call takes, and how wide, on both sides of the limits that a count of launches does not show, with 256 compute
units.  Runs without a GPU, against a recording stand-in for the runtime."""
import ctypes as C
import json
import sys

import pytest

from tests.bruteforce import ntt_primes
from tests.stubbed import DEV as d, Stubbed, run, u32, vp
from workloads.params import ParamSet

class _KernelStat(C.Structure):
    _fields_ = [("kernel_id", u32), ("launches", u32), ("total_ms", C.c_double), ("algo_bytes", C.c_double),
                ("work_items", C.c_double)]


# name -> log2 N, primes, special primes, primes of a digit
SETS = {"n8192_k3": (13, 3, 1, 1), "n8192_k4": (13, 4, 1, 1), "n4096_k2": (12, 2, 1, 1), "n16384_k6": (14, 6, 2, 2)}
TENSOR, SUMS = "ntt_inv_kernel<13, {}, LdInvTensor, StTens<false> >", "mul_sum_row_kernel<13, 8, 3, false>"
# set, call, its sizes -> the kernel among its launches that tells the routes apart
WANT = {
    # 7 summed rotations: pairs of units where 1.84 rounds of pairs are less than the rounds of one unit ...
    **{("n8192_k3", "sum", b): "ks_sum_row_kernel<13, 8, 1>" for b in (64, 192, 320)},
    **{("n8192_k3", "sum", b): "ks_sum_row_kernel<13, 8, 2>" for b in (107, 128, 193, 256, 321)},
    # ... with four digits from 5 rows on 4 compute units, launches of single transforms below
    ("n8192_k4", "sum", 51): "ks_sum_row_kernel<13, 8, 1>", ("n8192_k4", "sum", 52): "ks_sum_kernel<4, ",
    ("n8192_k4", "sum", 63): "ks_sum_kernel<4, ", ("n8192_k4", "sum", 64): "ks_sum_row_kernel<13, 8, 2>",
    **{("n4096_k2", "sum", b): "ks_sum_row_kernel<12, 8, 1>" for b in (64, 200, 400)},
    # the tensor product of no more rows than compute units on 1024 threads
    ("n8192_k3", "mul", 12): TENSOR.format(8), ("n8192_k3", "mul", 13): TENSOR.format(16),
    # transforms: rows in four parts up to a quarter of the compute units, in two up to half; inverse at N = 8192 in two up to
    # half and from one row per unit to 11/8, at N = 16384 in four up to a quarter
    **{("n8192_k3", "fwd", r): f"ntt_fwd_part_kernel<13, {p}, LdRowsU64, StU64>" for r, p in ((1, 2), (64, 2), (65, 1), (128, 1))},
    ("n8192_k3", "fwd", 129): "ntt_fwd_kernel<13, 8, LdRowsU64, StU64>",
    **{("n8192_k3", "inv", r): "ntt_inv_part_kernel<13, 1, LdInvU64, StInvU64>" for r in (1, 86, 128, 257, 352)},
    **{("n8192_k3", "inv", r): "ntt_inv_kernel<13, 8, LdInvU64, StInvU64>" for r in (129, 256, 353)},
    ("n4096_k2", "fwd", 64): "ntt_fwd_part_kernel<12, 2, LdRowsU64, StU64>", ("n4096_k2", "inv", 1): "ntt_inv_kernel<12, 8, LdInvU64, StInvU64>",
    ("n16384_k6", "inv", 64): "ntt_inv_part_kernel<14, 2, LdInvU64, StInvU64>", ("n16384_k6", "inv", 65): "ntt_inv_kernel<14, 16, LdInvU64, StInvU64>",
    # ... accumulators of summed rotations (8 and 16 rows a unit) up to an eighth, at N = 16384 alone up to a quarter
    **{("n8192_k3", "sum", b): "ntt_inv_part_kernel<13, 1, LdInvF64, StInvF64>" for b in (1, 4, 33, 41)},
    **{("n8192_k3", "sum", b): "ntt_inv_kernel<13, 8, LdInvF64, StInvF64>" for b in (5, 10, 32)},
    ("n16384_k6", "sum", 3): "ntt_inv_part_kernel<14, 2, LdInvF64, StInvF64>", ("n16384_k6", "sum", 5): "ntt_inv_kernel<14, 16, LdInvF64, StInvF64>",
    ("n16384_k6", "step", 2, 1): "ntt_inv_part_kernel<14, 2, LdInvF64, StInvF64>",
    # ... not where the results land on the rows that are read
    ("n8192_k3", "fwd_in_place", 12): "ntt_fwd_kernel<13, 8, LdRowsU64, StU64>",
    ("n8192_k3", "inv_in_place", 12): "ntt_inv_kernel<13, 8, LdInvU64, StInvU64>",
    # key switches at N = 16384: single transforms' launches while more than 5/16 of the compute units would idle in one round, 9/16 in two
    **{("n16384_k6", "sum", b): "ks_sum_kernel<3, " for b in (4, 20, 21, 33, 45)},
    **{("n16384_k6", "sum", b): "ks_wide_kernel<2>" for b in (22, 32, 46, 64, 80)},
    # ... in calls made alone as well (other limits beside a step's branches)
    **{("n16384_k6", "scores_rounds", b, 1): "ks_sum_kernel<3, " for b in (16, 17, 18, 19)}, ("n16384_k6", "scores_rounds", 16, 2): "ks_wide_kernel<2>",
    **{("n16384_k6", "context_ext", 16, c): "ks_sum_kernel<3, " for c in (1, 2, 3)}, ("n16384_k6", "context_ext", 19, 1): "ks_sum_kernel<3, ",
    # ... where relinearisations stay with them up to one round
    ("n16384_k6", "step", 16, 2): "ntt_inv_kernel<14, 16, LdInvKsInner<3>, StInvF64>",
    # operands: no more rows than compute units on 1024 threads; both kinds of rows in one launch up to two per unit
    ("n8192_k3", "extend", 18): "ntt_fwd_kernel<13, 8, LdMulExt<3>, StF64>",
    ("n8192_k3", "extend", 19): "ntt_fwd_kernel<13, 16, LdMulExt<3>, StF64>",
    ("n8192_k3", "extend", 36): "ntt_fwd_kernel<13, 16, LdMulExt<3>, StF64>",
    ("n8192_k3", "extend", 37): "ntt_fwd_kernel<13, 16, LdMulAux<3>, StF64>",
    ("n16384_k6", "extend", 4): "ntt_fwd_kernel<13, 8, LdHalf, StF64>",
    ("n16384_k6", "extend", 5): "ntt_fwd_kernel<13, 16, LdHalf, StF64>",
    # products of a step, beside its other branches, with more units idle than alone
    ("n8192_k3", "scores", 12, 4): "mul_row_kernel<13, 8, 3, true>", ("n8192_k3", "scores", 11, 4): TENSOR.format(16),
    ("n8192_k3", "mul", 48): TENSOR.format(16),
    # sums of products by the model of both routes
    **{("n8192_k3", "mul_sum", g, u): SUMS for g, u in ((3, 8), (16, 8), (4, 16), (8, 100))},
    **{("n8192_k3", "mul_sum", g, u): "ntt_inv_kernel<13, 8, LdInvTensorSum, StTens<false> >" for g, u in ((12, 4), (12, 8), (6, 8))},
    # with a transformed cache at N = 4096 up to 5/3 rows of (unit, prime) per compute unit, at N = 8192 never
    **{("n4096_k2", "context_ext", h, c): "mul_sum_row_kernel<12, 8, 2, true>" for h, c in ((17, 5), (85, 1), (12, 7))},
    **{("n4096_k2", "context_ext", h, c): "ntt_inv_kernel<12, 8, LdInvTensorSum, StTens<false> >" for h, c in ((43, 2), (86, 1), (11, 8))},
    ("n8192_k3", "context_ext", 1, 1): "ntt_inv_kernel<13, 8, LdInvTensorSum, StTens<false> >",
    # ... at N = 8192 product by product from 7/16 rows of (unit, prime) per compute unit to 7/8, in a step to 2/3 and not beside the longer chain
    ("n8192_k3", "step", 8, 3, 64): "mul_row_kernel<13, 8, 3, true>", ("n8192_k3", "step", 8, 3, 128): "ntt_inv_kernel<13, 8, LdInvTensorSum, StTens<false> >",
    ("n8192_k3", "step", 5, 5, 64): "ntt_inv_kernel<13, 8, LdInvTensorSum, StTens<false> >",
    **{("n8192_k3", "context_ext", h, c): "ntt_inv_kernel<13, 8, LdInvTensorSum, StTens<false> >" for h, c in ((15, 1), (11, 3), (12, 4))},
    **{("n8192_k3", "context_ext", h, c): "mul_row_kernel<13, 8, 3, true>" for h, c in ((16, 1), (2, 8), (8, 4))},
    # the context's key switches in parts, in a step until the scores' mod-ups have a row for every compute unit; at N = 16384 in one launch, up to half idle, where
    # the scores' take one launch (up to 3/8)
    **{("n8192_k3", op, 7, c): "ntt_fwd_part_kernel<13, 1, LdModup<false, 1>, StU64>" for op, c in (("context_ext", 3), ("context_ext", 4), ("step", 3))},
    **{("n8192_k3", op, 4, c): "ntt_inv_part_kernel<13, 1, LdInvF64, StInvF64>" for op, c in (("context_ext", 5), ("context_ext", 6), ("step", 5))},
    **{("n16384_k6", "step", h, c): "ks_wide_kernel<2>" for h, c in ((16, 3), (10, 2))}, ("n16384_k6", "step", 15, 2): "ks_sum_kernel<3, ",
    # a transformed cache at N = 16384: parts of one unit each (the fewest that are as fast), and of several
    **{("n16384_k6", "context_ext", h, c): "mul_row_kernel<13, 8, 0, true>" for h, c in ((1, 1), (1, 4), (2, 4), (3, 2), (16, 1))},
    **{("n16384_k6", "context_ext", h, c): "mul_sum_row_kernel<13, 8, 0, true>" for h, c in ((4, 4), (8, 3), (12, 2), (16, 3))},
}
# ... -> kernels that are not among them
NEVER = {
    **{("n16384_k6", "scores_rounds", b, 1): "ks_wide_kernel" for b in (16, 17, 18, 19)}, **{("n16384_k6", "context_ext", 16, c): "ks_wide_kernel" for c in (1, 2, 3)},
    ("n16384_k6", "context_ext", 19, 1): "ks_wide_kernel",
    ("n16384_k6", "scores_rounds", 16, 2): "ntt_inv_kernel<14, 16, LdInvKsInner<3>, StInvF64>",      # (its relinearisation)
    **{("n16384_k6", "step", h, c): "ks_wide_kernel" for h, c in ((16, 1), (17, 1), (17, 2), (19, 1), (9, 2))},
    **{("n16384_k6", "step", h, c): "ks_sum_kernel" for h, c in ((16, 2), (16, 3), (16, 5))},
    ("n8192_k3", "step", 7, 4): "ntt_fwd_part_kernel", ("n8192_k3", "step", 4, 6): "ntt_inv_part_kernel", ("n16384_k6", "step", 3, 1): "ntt_inv_part_kernel",
}


def _profile(lib, ctx, call):
    """kernel classes the library's own timing names for `call`: [[name, launches, items], ...]"""
    stats, n = (_KernelStat * 64)(), u32()
    lib.lib.cg_kernel_name.restype = C.c_char_p
    assert lib.lib.cg_profile_begin(ctx, u32(256)) == 0
    assert call() == 0
    assert lib.lib.cg_profile_end(ctx, stats, u32(64), C.byref(n)) == 0
    return [[lib.lib.cg_kernel_name(s.kernel_id).decode(), s.launches, s.work_items] for s in stats[:n.value]]


def _launches(lib):
    got = {}
    gs, keys, out = (u32 * 16)(*range(3, 35, 2)), (vp * 256)(*[1 << 20] * 256), vp(1 << 40)   # (no output overlaps its input)
    for name, (log2n, k, nsp, alpha) in SETS.items():
        p = ntt_primes(1 << 50, 2 << log2n, k + nsp)
        ctx = lib.create(ParamSet(name, log2n, q=tuple(p[:k]), p=tuple(p[k:]), alpha=alpha))
        calls = {"mul": lambda b: lib.lib.cg_mul(ctx, None, d, d, out, u32(b), u32(1), d),
                 "mul_sum": lambda g, u: lib.lib.cg_mul_sum(ctx, None, d, d, out, u32(g), u32(u), d),
                 "sum": lambda b: lib.lib.cg_rotate_sum_hoisted(ctx, None, d, u32(7), gs, keys, out, u32(b), d),
                 "extend": lambda n: lib.lib.cg_cache_extend(ctx, None, d, u32(n), u32(1), u32(1), out),
                 **{name + at: lambda r, f=f, to=to: getattr(lib.lib, f)(ctx, None, d, to, (u32 * r)(*[i % k for i in range(r)]), u32(r))
                    for name, f in (("fwd", "cg_ntt_forward"), ("inv", "cg_ntt_inverse")) for at, to in (("", out), ("_in_place", d))},
                 "scores_rounds": lambda h, c: lib.lib.cg_decode_scores_hoisted(
                     ctx, None, d, d, None, u32(h), u32(c), u32(c), u32(64), u32(3), d, keys, out, d),
                 "scores": lambda h, c: lib.lib.cg_decode_scores(ctx, None, d, d, u32(h), u32(c), u32(c), u32(64), d, keys, out, d),
                 "context_ext": lambda h, c: lib.lib.cg_decode_context_hoisted(
                     ctx, None, d, d, d, u32(h), u32(c), u32(c), u32(64), u32(3), 1, d, keys, out, d),
                 "step": lambda h, c, d2=64: lib.lib.cg_decode_step_hoisted(
                     ctx, None, d, d, d, d, u32(h), u32(c), u32(c + 1), u32(d2), u32(c * (1 << log2n) // d2 - 1), d, d, d, u32(3), keys, u32(3),
                     1, keys, out, out, d)}
        for s, op, *sizes in {**WANT, **NEVER}:
            if s == name:
                got[" ".join(map(str, (s, op, *sizes)))] = lib.kernels(lambda: calls[op](*sizes))
        if name == "n8192_k3":
            got["profile"] = _profile(lib, ctx, lambda: lib.lib.cg_prefill_av_hoisted(ctx, None, d, d, u32(3), u32(64), 1, d, keys,
                                                                                      out, d))
        assert lib.lib.cg_destroy(ctx) == 0
    return got


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    return run(__file__, tmp_path_factory.mktemp("stub"))


@pytest.mark.parametrize("case", WANT, ids=lambda c: " ".join(map(str, c)))
def test_kernel(launches, case):
    names = [k[0] for k in launches[" ".join(map(str, case))]]
    assert any(n.startswith(WANT[case]) for n in names), names


@pytest.mark.parametrize("case", NEVER, ids=lambda c: " ".join(map(str, c)))
def test_other_kernels(launches, case):
    names = [k[0] for k in launches[" ".join(map(str, case))]]
    assert names and not any(n.startswith(NEVER[case]) for n in names), names


def test_copies_are_not_timed_as_sums(launches):
    """A V of three heads: a copy of every head's V, rotated copies, products, one relinearisation; nothing is added up"""
    classes = {name: (n, items) for name, n, items in launches["profile"]}
    assert classes["copy"] == (1, 3)
    assert "add" not in classes


if __name__ == "__main__":
    print(json.dumps(_launches(Stubbed(*sys.argv[1:]))))
