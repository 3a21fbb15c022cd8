"""What a server built on this library computes, as a set of sized calls.

The parameter sets are the presets of `workloads.params`; shapes are those of the benchmark
configurations (12 heads of 64 at N = 8192, 512 tokens of context, a prompt of 128 tokens, 16 heads at
N = 16384) and of what lies around them: one sequence with one head, short and long caches, odd head
counts, odd batches.  Ciphertexts, keys and plaintexts are uniform residues, which is what fresh
ciphertexts and keys look like to every kernel.  All results are residues, so they compare exactly.

kinds
  ntt            cg_ntt_forward / cg_ntt_inverse over a stack of ring rows
  mul_relin      ciphertext products with relinearisation, one call per batch
  append_prompt  a prompt's tokens appended to the K and V caches of all heads, one call per token
  step           one generated token's attention in one call, all four forms
  prompt_scores  Q K^T of a prompt over its diagonals, then the compaction sent to the client
  prompt_context A V of a prompt
  project        one token's ciphertext times the plaintext matrices of a layer's projections
"""
import torch

import paper_2602_08798_amd as P
from workloads import PRESETS

_CONTEXTS = {}


def _context(params):
    """A program holds one context per parameter set for as long as it runs."""
    if params not in _CONTEXTS:
        _CONTEXTS[params] = P.Context(PRESETS[params])
    return _CONTEXTS[params]


def listed():
    return [
        # one fresh ciphertext of the small ring taken back to coefficients: the smallest call there is
        {"name": "ntt_inverse_one_ct", "kind": "ntt", "params": "C1", "rows": 4, "inverse": True},
        # a whole cache's worth of rows in one call
        {"name": "ntt_forward_16384_rows", "kind": "ntt", "params": "C2", "rows": 16384, "inverse": False},
        # configuration C1: 16 independent products at N = 4096
        {"name": "mul_relin_16_n4096", "kind": "mul_relin", "params": "C1", "batch": 16},
        # a saturating batch of products at N = 8192 (several sequences or layers together)
        {"name": "mul_relin_768_n8192", "kind": "mul_relin", "params": "C2", "batch": 768},
        # configuration C3's appends: 128 prompt tokens into 12 K and 12 V caches
        {"name": "append_prompt_128x24", "kind": "append_prompt", "params": "C3", "heads": 12, "tokens": 128, "d2": 64},
        # configuration C2's shape: one head whose single cache ciphertext is being filled (token 100 of 128)
        {"name": "step_one_head", "kind": "step", "params": "C2", "heads": 1, "n_cts": 1, "d2": 64, "tau": 100,
         "hoisted": True, "ext": False},
        # configuration C4 with the rotate-and-add chains of the textbook form: 13 rotation keys, plain cache
        {"name": "step_12_heads_chain", "kind": "step", "params": "C4", "heads": 12, "n_cts": 4, "d2": 64, "tau": 512,
         "hoisted": False, "ext": False},
        # configuration C4 in the form bench.py headlines: rounds of rotations, transformed copy of the cache
        {"name": "step_12_heads", "kind": "step", "params": "C4", "heads": 12, "n_cts": 4, "d2": 64, "tau": 512,
         "hoisted": True, "ext": True},
        # configuration C5: 16 heads at N = 16384, token 515 goes into the third ciphertext of every cache
        {"name": "step_16_heads_n16384", "kind": "step", "params": "C5", "heads": 16, "n_cts": 3, "d2": 64, "tau": 515,
         "hoisted": True, "ext": False},
        # configuration C3: Q K^T of 12 heads, 128 diagonals each, and their compaction
        {"name": "prompt_scores_12_heads", "kind": "prompt_scores", "params": "C3", "heads": 12, "d2": 64},
        # configuration C3: A V of 12 heads
        {"name": "prompt_context_12_heads", "kind": "prompt_context", "params": "C3", "heads": 12, "d2": 64},
        # one token times the 36 matrices (768 x 64) of a layer's Q, K and V projections
        {"name": "project_36_matrices", "kind": "project", "params": "C2", "units": 36, "n_diag": 8, "d2": 64},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["ntt", "mul_relin", "append_prompt", "step", "step", "step", "prompt_scores",
                       "prompt_context", "project"])
    params = rng.choice(["C1", "C2", "C2", "C5"])
    case = {"kind": kind, "params": params}
    if kind == "ntt":
        case.update(rows=_log_int(rng, 1, 8192 if params == "C5" else 16384), inverse=rng.random() < 0.5)
    elif kind == "mul_relin":
        case.update(batch=_log_int(rng, 1, 96 if params == "C5" else 768))
    elif kind == "append_prompt":
        case.update(heads=rng.randint(1, 16), tokens=_log_int(rng, 1, 128), d2=rng.choice([32, 64, 128]))
    elif kind == "step":
        d2 = rng.choice([32, 64, 64, 128])
        n_cts = _log_int(rng, 1, 4 if params == "C5" else 8)
        blocks = PRESETS[params].n // d2
        # the new token lands in the last ciphertext the products read, or opens the next one
        tau = n_cts * blocks - rng.randint(0, blocks)
        case.update(heads=rng.randint(1, 16), n_cts=n_cts, d2=d2, tau=tau, hoisted=rng.random() < 0.67,
                    ext=rng.random() < 0.5)
    elif kind == "project":
        case.update(units=_log_int(rng, 1, 48), n_diag=rng.choice([2, 4, 8, 16]), d2=64)
    else:
        if params == "C5":
            case["params"] = "C2"
        case.update(heads=rng.randint(1, 12), d2=64)
    return case


# bits per round of the folding sums, as in workloads.configs.C4_ROUND_BITS
ROUND_BITS = 3


class _Draws:
    """Uniform residues on the GPU from one seed."""

    def __init__(self, prm, seed):
        self.prm = prm
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def residues(self, primes, *lead):
        """[*lead][len(primes)][n], row i below primes[i]"""
        out = torch.empty(*lead, len(primes), self.prm.n, dtype=torch.int64, device="cuda")
        for i, p in enumerate(primes):
            out[..., i, :] = torch.randint(0, int(p), (*lead, self.prm.n), generator=self.g, device="cuda")
        return out

    def cts(self, *lead):
        return self.residues(self.prm.q, *lead, 2)

    def keys(self, ctx, count):
        raw = self.residues(list(self.prm.q) + list(self.prm.p), count, self.prm.dnum, 2)
        return [ctx.ksk_prepare(raw[i]) for i in range(count)]

    def plains(self, ctx, count):
        pt = torch.randint(0, self.prm.t, (count, self.prm.n), generator=self.g, device="cuda")
        return ctx.plain_prepare(pt)


def _bits(x):
    return x.bit_length() - 1


def prepare(case, seed):
    prm = PRESETS[case["params"]]
    ctx = _context(case["params"])
    r = _Draws(prm, seed)
    n = prm.n
    s = {"case": case, "ctx": ctx}
    kind = case["kind"]
    if kind == "ntt":
        primes = list(prm.q) if case["rows"] % prm.k == 0 else list(prm.q) + list(prm.p)
        # row i modulo prime i mod period: stacked ciphertexts, or stacked switching-key rows
        rows = case["rows"]
        full = r.residues(primes, -(-rows // len(primes)))
        s["idx"] = [i % len(primes) for i in range(rows)]
        s["x"] = full.view(-1, n)[:rows].contiguous()
    elif kind == "mul_relin":
        s["a"], s["b"] = r.cts(case["batch"]), r.cts(case["batch"])
        s["rlk"] = r.keys(ctx, 1)[0]
    elif kind == "append_prompt":
        blocks = n // case["d2"]
        caches = 2 * case["heads"]
        s["stride"] = -(-case["tokens"] // blocks)
        s["rows"] = r.cts(case["tokens"], caches)
        s["cache"] = torch.zeros(caches * s["stride"], 2, prm.k, n, dtype=torch.int64, device="cuda")
        s["masks"] = r.plains(ctx, min(blocks, case["tokens"]))
    elif kind == "step":
        H, C, d2 = case["heads"], case["n_cts"], case["d2"]
        s["stride"] = stride = C + 1
        s["q"], s["a"], s["rows"] = r.cts(H), r.cts(H * C), r.cts(2 * H)
        s["cache"] = r.cts(2 * H * stride)
        s["masks"] = r.plains(ctx, n // d2)
        s["rlk"] = r.keys(ctx, 1)[0]
        if case["hoisted"]:
            n_fold, n_block = (len(ctx.round_galois(w, d2, ROUND_BITS)) for w in (0, 1))
        else:
            n_fold, n_block = _bits(d2), _bits(n // d2)
        s["fold"], s["block"] = r.keys(ctx, n_fold), r.keys(ctx, n_block)
        s["ext"] = None
        if case["ext"]:
            s["ext"] = ctx.empty_ext(2 * H * stride)
            ctx.cache_extend(s["cache"], 2 * H, stride, stride, s["ext"])
        s["scores"], s["context"] = ctx.empty_ct(H, C), ctx.empty_ct(H)
    elif kind in ("prompt_scores", "prompt_context"):
        H, d2 = case["heads"], case["d2"]
        m = n // d2
        s["rlk"] = r.keys(ctx, 1)[0]
        s["copies"] = r.keys(ctx, m - 1)
        if kind == "prompt_scores":
            s["q"], s["k"] = r.cts(H), r.cts(H)
            s["fold"] = r.keys(ctx, len(ctx.round_galois(0, d2, ROUND_BITS)))
            s["right"] = r.keys(ctx, _bits(min(d2, m // 2)))
            s["mask0"] = r.plains(ctx, 1)
        else:
            s["a"], s["v"] = r.cts(H * m), r.cts(H)
    elif kind == "project":
        s["x"] = r.cts(1)
        s["diags"] = r.plains(ctx, case["units"] * case["n_diag"])
        s["copies"] = r.keys(ctx, case["n_diag"] - 1)
        s["block"] = r.keys(ctx, len(ctx.round_galois(1, case["d2"], ROUND_BITS)))
    else:
        raise ValueError(kind)
    return s


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "ntt":
        return ctx.ntt_inverse(s["x"], s["idx"]) if case["inverse"] else ctx.ntt_forward(s["x"], s["idx"])
    if kind == "mul_relin":
        return ctx.mul_relin(s["a"], s["b"], s["rlk"], case["batch"])
    if kind == "append_prompt":
        for tau in range(case["tokens"]):
            ctx.kv_append(s["cache"], s["stride"], 2 * case["heads"], tau, s["rows"][tau], s["masks"], case["d2"])
        return s["cache"]
    if kind == "step":
        if case["hoisted"]:
            ctx.decode_step_hoisted(s["q"], s["a"], s["cache"], case["heads"], case["n_cts"], s["stride"], case["d2"],
                                    case["tau"], s["rows"], s["masks"], s["rlk"], ROUND_BITS, s["fold"], ROUND_BITS,
                                    s["block"], scores=s["scores"], context=s["context"], cache_ext=s["ext"],
                                    sum_before_scaling=True)
        else:
            ctx.decode_step(s["q"], s["a"], s["cache"], case["heads"], case["n_cts"], s["stride"], case["d2"],
                            case["tau"], s["rows"], s["masks"], s["rlk"], s["fold"], s["block"], scores=s["scores"],
                            context=s["context"], cache_ext=s["ext"])
        return {"scores": s["scores"], "context": s["context"], "cache": s["cache"]}
    if kind == "prompt_scores":
        out = ctx.prefill_qk_hoisted(s["q"], s["k"], case["heads"], case["d2"], s["rlk"], s["fold"], s["copies"],
                                     fold_round_bits=ROUND_BITS)
        return {"diagonals": out, "packed": ctx.prefill_repack(out, case["heads"], case["d2"], s["mask0"], s["right"])}
    if kind == "prompt_context":
        return ctx.prefill_av_hoisted(s["a"], s["v"], case["heads"], case["d2"], s["rlk"], s["copies"],
                                      sum_before_scaling=True)
    return ctx.cpvm_hoisted(s["x"], s["diags"], case["units"], case["n_diag"], case["d2"], s["copies"], s["block"],
                            block_round_bits=ROUND_BITS)


def _rounds(bits):
    """Rotations of each round of a folding sum over `bits` generators."""
    if not bits:
        return []
    n = -(-bits // ROUND_BITS)
    lo, extra = divmod(bits, n)
    return [(1 << (lo + (1 if i < extra else 0))) - 1 for i in range(n)]


class _Count:
    """Rows that cross memory once, row transforms, and modular products per coefficient."""

    def __init__(self, prm):
        self.k, self.L, self.KL, self.dnum = prm.k, prm.k + prm.nsp, 2 * prm.k + 1, prm.dnum
        self.n, self.log2n = prm.n, prm.log2n
        self.rows = self.transforms = self.products = 0

    def cts(self, count):
        self.rows += 2 * self.k * count

    def keys(self, count):
        self.rows += 2 * self.dnum * self.L * count

    def mul(self, operands, units, results):
        """`operands` ciphertexts transformed, `units` tensor products, `results` scaled results"""
        self.transforms += self.KL * (2 * operands + 3 * results)
        self.products += self.KL * (4 * units + 3 * results) + 3 * results * (self.k * self.k + 2 * self.KL)

    def switch(self, units, rotations=1, decompose=True):
        """key switches of `units` ciphertexts, `rotations` inner products summed in each"""
        self.transforms += units * ((self.dnum * self.L if decompose else 0) + 2 * self.L)
        self.products += units * 2 * (rotations * self.dnum * self.L + 2 * self.k)

    def result(self):
        # a butterfly is a modular product (8 operations in FP64, a fused multiply-add counted twice)
        # and two sums
        return {"bytes": 8 * self.n * self.rows,
                "flops": 10 * self.transforms * self.n // 2 * self.log2n + 8 * self.products * self.n}


def work(case):
    prm = PRESETS[case["params"]]
    c = _Count(prm)
    n, k, kind = prm.n, prm.k, case["kind"]
    if kind == "ntt":
        c.rows += 2 * case["rows"]
        c.transforms += case["rows"]
    elif kind == "mul_relin":
        b = case["batch"]
        c.cts(3 * b)
        c.keys(1)
        c.mul(2 * b, b, b)
        c.switch(b)
    elif kind == "append_prompt":
        caches, tokens = 2 * case["heads"], case["tokens"]
        c.cts(caches * tokens + caches * -(-tokens // (n // case["d2"])))
        c.rows += k * min(tokens, n // case["d2"])
        # the appends are linear: one transform of each row and one of each cache ciphertext would do
        c.transforms += 2 * k * caches * (tokens + 1)
        c.products += 2 * k * caches * tokens
    elif kind == "step":
        H, C, d2 = case["heads"], case["n_cts"], case["d2"]
        fold, block = _bits(d2), _bits(n // d2)
        opens = case["tau"] % (n // d2) == 0
        c.cts(H + H * C + 2 * H + H * C + H + 2 * H * (1 if opens else 2))    # q, a, rows, scores, context, cache
        c.rows += 2 * (c.KL if case["ext"] else k) * 2 * H * C                # the cache the products read
        c.rows += k
        c.transforms += 2 * k * 2 * H * 2                                     # append
        if case["ext"]:
            c.transforms += 2 * c.KL * 2 * H
            c.rows += 2 * c.KL * 2 * H
        read = 0 if case["ext"] else H * C
        c.mul(H + read, H * C, H * C)
        c.mul(H * C + read, H * C, H if case["hoisted"] else H * C)
        c.switch(H * C + H)
        rf, rb = (_rounds(fold), _rounds(block)) if case["hoisted"] else ([1] * fold, [1] * block)
        for x in rf:
            c.switch(H * C, x)
        for x in rb:
            c.switch(H, x)
        c.keys(1 + sum(rf) + sum(rb))
    elif kind in ("prompt_scores", "prompt_context"):
        H, d2 = case["heads"], case["d2"]
        m = n // d2
        c.keys(1 + m - 1)
        c.switch(H)                                                           # decomposition shared by the copies
        c.switch(H * (m - 2), decompose=False)
        if kind == "prompt_scores":
            w = min(d2, m // 2)
            rf = _rounds(_bits(d2))
            c.keys(sum(rf) + _bits(w))
            c.cts(2 * H + H * m + H * m // w)
            c.rows += k
            c.mul(H + H * m, H * m, H * m)
            c.switch(H * m)
            for x in rf:
                c.switch(H * m, x)
            c.transforms += 2 * 2 * k * H * m
            c.products += 2 * k * H * m
            c.switch(H * m - H * m // w)
        else:
            c.cts(H * m + H + H)
            c.mul(2 * H * m, H * m, H)
            c.switch(H)
    else:
        units, nd = case["units"], case["n_diag"]
        rb = _rounds(_bits(n // case["d2"]))
        c.cts(1 + units)
        c.rows += units * nd * k
        c.keys(nd - 1 + sum(rb))
        c.switch(1)
        c.switch(nd - 2, decompose=False)
        c.transforms += 2 * k * (nd + units)
        c.products += 2 * k * nd * units
        for x in rb:
            c.switch(units, x)
    return c.result()


def tolerance(case):
    return "exact"
