"""Attention calls of few units, whose rounds of summed rotations take the mod-down before them in the mod-up's loader and beside the sums, against the
same product, relinearisation and summed rotations as calls of their own, bit for bit (those are compared with the oracle elsewhere).  Numbers of units on
both sides of the rule's limits (256 compute units) and of where rows go from quarters to halves; rounds of one to four bits (1 to 15 rotations);
uniform residues and the largest ones.  The same for chains of single rotations."""
import pytest

pytestmark = pytest.mark.gpu

from workloads import PRESETS
from workloads.params import ParamSet

from .bruteforce import ntt_primes
from .test_gpu_parity import say

_P, _P12 = ntt_primes(1 << 50, 2 << 13, 3), ntt_primes(1 << 50, 2 << 12, 4)
_set = lambda log2n, k, p: ParamSet(f"n{1 << log2n}_k{k}_joined", log2n, q=tuple(p[:k]), p=tuple(p[k:k + 1]), alpha=1)
SETS = {**PRESETS, "k1": _set(13, 1, _P), "k2": _set(13, 2, _P), "n4096_k1": _set(12, 1, _P12), "n4096_k3": _set(12, 3, _P12)}
_state = {}


def _residues(primes, n, largest, *lead):
    import torch
    g = _state.setdefault("generator", torch.Generator(device="cuda").manual_seed(78))
    out = torch.empty(*lead, len(primes), n, dtype=torch.int64, device="cuda")
    for i, p in enumerate(primes):
        out[..., i, :] = int(p) - 1 if largest else torch.randint(0, int(p), (*lead, n), generator=g, device="cuda")
    return out


def _ctx(name, largest):
    import paper_2602_08798_amd as P
    if (name, largest) not in _state:
        prm = SETS[name]
        ctx = P.Context(prm)
        _state[name, largest] = ctx, [ctx.ksk_prepare(_residues(list(prm.q) + list(prm.p), prm.n, largest, prm.dnum, 2)) for _ in range(3)]
    return _state[name, largest]


def _rounds(bits, w):
    n = -(-bits // w)
    lo, extra = divmod(bits, n)
    return [(1 << (lo + (r < extra))) - 1 for r in range(n)]


@pytest.mark.parametrize("name,units,d2,w,largest", [
    ("C2", 1, 64, 3, False), ("C2", 1, 2, 3, False), ("C2", 2, 128, 1, False), ("C2", 3, 32, 2, True), ("C2", 5, 256, 4, False), ("C2", 6, 64, 3, False),
    ("C1", 1, 64, 3, True), ("C1", 10, 64, 3, False), ("C1", 11, 32, 3, False), ("C1", 21, 16, 4, True), ("C1", 22, 64, 3, False),
    ("k1", 3, 64, 3, False), ("k1", 32, 16, 2, False),
    ("C2", 2, 64, 4, True), ("k1", 8, 64, 3, True), ("k2", 1, 64, 3, True), ("k2", 4, 32, 4, False), ("n4096_k1", 1, 64, 3, False), ("n4096_k1", 37, 16, 3, True),
    ("n4096_k3", 2, 64, 3, False), ("n4096_k3", 10, 32, 4, True)])
def test_joined_rounds(name, units, d2, w, largest):
    import torch
    say(f"joined rounds {name}: {units} units, d2 = {d2}, {w} bits, largest {largest}")
    prm = SETS[name]
    ctx, keys = _ctx(name, largest)
    x, y = _residues(prm.q, prm.n, largest, units, 2), _residues(prm.q, prm.n, largest, units, 2)
    slots, blocks = d2.bit_length() - 1, (prm.n // d2).bit_length() - 1
    for which, bits in ((0, slots), (1, blocks)):
        gs = ctx.round_galois(which, d2, w)
        used = [keys[1 + i % 2] for i in range(len(gs))]
        want, at = ctx.relin(ctx.mul(x, y, units), keys[0], units), 0
        for n in _rounds(bits, w):
            want = ctx.rotate_sum_hoisted(want, gs[at:at + n], used[at:at + n], units)
            at += n
        assert at == len(gs)
        got = (ctx.decode_context_hoisted if which else ctx.decode_scores_hoisted)(x, y, units, 1, d2, w, keys[0], used)
        assert torch.equal(got.view(-1), want.view(-1)), (name, units, which)


@pytest.mark.parametrize("name,units,d2,largest", [("C2", 1, 2, False), ("C2", 3, 64, True), ("C2", 21, 128, False), ("C2", 22, 64, False), ("C1", 1, 64, True),
                                                   ("C1", 42, 32, False), ("C1", 43, 64, False), ("C1", 64, 16, False), ("C1", 65, 64, False), ("k1", 5, 64, False),
                                                   ("k2", 1, 64, False), ("k2", 34, 16, True), ("n4096_k1", 3, 64, True), ("n4096_k1", 117, 16, False), ("n4096_k3", 1, 64, False),
                                                   ("n4096_k3", 32, 16, True)])
def test_joined_chain(name, units, d2, largest):
    import torch
    say(f"joined chain {name}: {units} units, d2 = {d2}, largest {largest}")
    prm = SETS[name]
    ctx, keys = _ctx(name, largest)
    x, y = _residues(prm.q, prm.n, largest, units, 2), _residues(prm.q, prm.n, largest, units, 2)
    slots, blocks = d2.bit_length() - 1, (prm.n // d2).bit_length() - 1
    step = lambda i: pow(3, 1 << i, 2 * prm.n)
    for which, gs in ((0, [step(i) for i in range(slots)]), (1, [step(slots + i) for i in range(blocks - 1)] + [2 * prm.n - 1])):
        used = [keys[1 + i % 2] for i in range(len(gs))]
        want = ctx.relin(ctx.mul(x, y, units), keys[0], units)
        for g, key in zip(gs, used):
            want = ctx.rotate(want, g, key, units, accumulate=True)
        got = (ctx.decode_context if which else ctx.decode_scores)(x, y, units, 1, d2, keys[0], used)
        assert torch.equal(got.view(-1), want.view(-1)), (name, units, which)


# ... and where no relinearisation is ahead of the chain
@pytest.mark.parametrize("name,units", [("C2", 1), ("C2", 20), ("C1", 1), ("C1", 30)])
def test_joined_chain_of_a_projection(name, units):
    import torch
    say(f"joined chain of a projection {name}: {units} units")
    prm, d2 = SETS[name], 64
    ctx, keys = _ctx(name, False)
    x, zero = _residues(prm.q, prm.n, False, 1, 2), []
    diags = ctx.plain_prepare(torch.randint(0, prm.t, (units, prm.n), device="cuda"))
    gs = ctx.round_galois(1, d2, 1)
    used = [keys[i % 3] for i in range(len(gs))]
    want = ctx.mul_plain(x.expand(units, -1, -1, -1).contiguous(), diags, units, plain_stride=1)
    for g, key in zip(gs, used):
        want = ctx.rotate(want, g, key, units, accumulate=True)
    got = ctx.cpvm(x, diags, units, 1, d2, zero, used)
    assert torch.equal(got.view(-1), want.view(-1)), (name, units)
