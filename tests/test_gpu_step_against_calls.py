"""The one-call decode step against the same work as calls made alone, bit for bit.  A step chooses the routes of its products and key
switches, and the order of its branches, by what runs beside them; a call made alone has nothing beside it.  Shapes on both sides of the
step's limits (256 compute units); the calls made alone are compared with the oracle elsewhere."""
import pytest

pytestmark = pytest.mark.gpu

from workloads import PRESETS

from .test_gpu_parity import say

# parameters, heads, ciphertexts, d2, transformed cache
SHAPES = [
    # which branch runs on the caller's stream: few rows of the scores, both chains' rows 5/4 of the compute units, as many key switches in both
    ("C2", 8, 7, 64, False), ("C2", 9, 5, 64, False), ("C2", 16, 2, 64, True), ("C2", 11, 3, 64, True), ("C2", 6, 3, 128, False), ("C1", 4, 4, 64, False),
    ("C1", 4, 4, 128, True),
    # sums with a transformed cache product by product, up to 2/3 of the compute units and not beside the longer chain
    ("C2", 2, 8, 64, True), ("C2", 5, 5, 64, True), ("C2", 8, 3, 128, True),
    # the context's rows in parts, until the scores' mod-ups have a row for every compute unit
    ("C2", 7, 3, 64, False), ("C2", 7, 4, 64, False), ("C2", 4, 5, 64, False), ("C5", 2, 1, 64, False), ("C5", 3, 1, 64, True),
    # whole units in one launch at N = 16384: the scores' from 20 units on, the context's from 16 heads on where the scores' are
    ("C5", 9, 2, 64, False), ("C5", 10, 2, 64, False), ("C5", 16, 1, 64, True), ("C5", 16, 2, 64, False),
]
_state = {}


def _residues(primes, n, *lead):
    import torch
    g = _state.setdefault("generator", torch.Generator(device="cuda").manual_seed(77))
    out = torch.empty(*lead, len(primes), n, dtype=torch.int64, device="cuda")
    for i, p in enumerate(primes):
        out[..., i, :] = torch.randint(0, int(p), (*lead, n), generator=g, device="cuda")
    return out


def _ctx(name):
    import paper_2602_08798_amd as P
    if name not in _state:
        prm = PRESETS[name]
        ctx = P.Context(prm)
        qp = list(prm.q) + list(prm.p)
        _state[name] = ctx, [ctx.ksk_prepare(_residues(qp, prm.n, prm.dnum, 2)) for _ in range(4)]
    return _state[name]


@pytest.mark.parametrize("name,heads,n_cts,d2,copy", SHAPES)
def test_step_and_calls_made_alone(name, heads, n_cts, d2, copy):
    import torch
    say(f"step against calls {name}: {heads} heads, {n_cts} ciphertexts, d2 = {d2}, transformed copy {copy}")
    prm = PRESETS[name]
    ctx, keys = _ctx(name)
    n, bits, stride = prm.n, 3, n_cts + 1
    ct = lambda *lead: _residues(prm.q, n, *lead, 2)
    q, a, rows, cache = ct(heads), ct(heads * n_cts), ct(2 * heads), ct(2 * heads * stride)
    masks = ctx.plain_prepare(torch.randint(0, prm.t, (n // d2, n), device="cuda"))
    fold, block = ([keys[1 + i % 3] for i in range(len(ctx.round_galois(which, d2, bits)))] for which in (0, 1))
    tau = n_cts * (n // d2) - 1                        # into the last ciphertext that the products read
    extended = lambda x: ctx.cache_extend(x, 2 * heads, stride, stride, ctx.empty_ext(2 * heads * stride)) if copy else None

    own = cache.clone()
    ctx.kv_append(own, stride, 2 * heads, tau, rows, masks, d2)
    ext = extended(own)
    half = heads * stride
    if copy:
        kext = ext.view(2 * half, -1)
        sides = dict(kext=kext[:half].contiguous()), dict(vext=kext[half:].contiguous())
        kc = vc = None
    else:
        sides, (kc, vc) = ({}, {}), (own[:half], own[half:])
    scores = ctx.decode_scores_hoisted(q, kc, heads, n_cts, d2, bits, keys[0], fold, cache_stride_cts=stride, **sides[0])
    context = ctx.decode_context_hoisted(a, vc, heads, n_cts, d2, bits, keys[0], block, cache_stride_cts=stride, sum_before_scaling=True,
                                         **sides[1])

    ext = extended(cache)
    got_scores, got_context = ctx.decode_step_hoisted(q, a, cache, heads, n_cts, stride, d2, tau, rows, masks, keys[0], bits, fold, bits,
                                                      block, cache_ext=ext, sum_before_scaling=True)
    torch.cuda.synchronize()
    assert torch.equal(cache, own)
    assert torch.equal(got_scores.view(-1), scores.view(-1))
    assert torch.equal(got_context.view(-1), context.view(-1))


# chains of single rotations: a context that takes the mod-downs in its mod-ups beside scores of a mod-up row for every unit, which it has two switches or
# more to do than; both branches of few units; neither
CHAINS = [("C2", 12, 4, 32), ("C2", 3, 4, 64), ("C2", 10, 3, 64), ("C1", 11, 4, 32), ("C1", 4, 4, 64)]


@pytest.mark.parametrize("name,heads,n_cts,d2", CHAINS)
def test_step_of_chains_and_calls_made_alone(name, heads, n_cts, d2):
    import torch
    say(f"step of chains against calls {name}: {heads} heads, {n_cts} ciphertexts, d2 = {d2}")
    prm = PRESETS[name]
    ctx, keys = _ctx(name)
    n, stride = prm.n, n_cts + 1
    ct = lambda *lead: _residues(prm.q, n, *lead, 2)
    q, a, rows, cache = ct(heads), ct(heads * n_cts), ct(2 * heads), ct(2 * heads * stride)
    masks = ctx.plain_prepare(torch.randint(0, prm.t, (n // d2, n), device="cuda"))
    fold, block = ([keys[1 + i % 3] for i in range(m.bit_length() - 1)] for m in (d2, n // d2))
    tau = n_cts * (n // d2) - 1

    own = cache.clone()
    ctx.kv_append(own, stride, 2 * heads, tau, rows, masks, d2)
    scores = ctx.decode_scores(q, own[:heads * stride], heads, n_cts, d2, keys[0], fold, cache_stride_cts=stride)
    context = ctx.decode_context(a, own[heads * stride:], heads, n_cts, d2, keys[0], block, cache_stride_cts=stride)
    got_scores, got_context = ctx.decode_step(q, a, cache, heads, n_cts, stride, d2, tau, rows, masks, keys[0], fold, block)
    torch.cuda.synchronize()
    assert torch.equal(cache, own)
    assert torch.equal(got_scores.view(-1), scores.view(-1))
    assert torch.equal(got_context.view(-1), context.view(-1))
