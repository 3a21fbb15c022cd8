"""One-call decode steps of two contexts: issued by two threads on two streams, and captured while the other context
runs steps of its own.  Every result must be what the context computes alone."""
import sys
import threading

import pytest

pytestmark = pytest.mark.gpu

from workloads import PRESETS, Stream, pseudo_ciphertexts, pseudo_switch_key


def say(msg):
    print(f"[gpu-two-contexts] {msg}", flush=True)
    sys.stdout.flush()


class Step:
    """a step that opens a new cache ciphertext (three branches; repeating it changes nothing)"""

    def __init__(self, preset, seed):
        import numpy as np
        import torch
        import paper_2602_08798_amd as P
        self.torch, prm = torch, PRESETS[preset]
        self.ctx = ctx = P.Context(prm)
        n, self.d2, self.heads = prm.n, 64, 3
        qp = list(prm.q) + list(prm.p)
        ct = lambda i, count: P.to_device(pseudo_ciphertexts(Stream(seed, i), prm.q, n, count))
        key = lambda i: ctx.ksk_prepare(P.to_device(pseudo_switch_key(Stream(seed, 50 + i), qp, n, prm.dnum)))
        self.q, self.a, self.rows, self.cache = ct(1, 3), ct(2, 3), ct(3, 6), ct(4, 12)
        pt = np.random.default_rng(seed).integers(0, prm.t, (1, n), dtype=np.uint64)
        self.masks, self.rlk = ctx.plain_prepare(P.to_device(pt)), key(0)
        some = [key(1 + i) for i in range(3)]
        self.keys = [[some[i % 3] for i in range(len(ctx.round_galois(w, self.d2, 3)))] for w in (0, 1)]
        self.tau = n // self.d2
        self.scores, self.context = ctx.empty_ct(3, 1), ctx.empty_ct(3)
        torch.cuda.synchronize()

    def __call__(self):
        self.ctx.decode_step_hoisted(self.q, self.a, self.cache, 3, 1, 2, self.d2, self.tau, self.rows, self.masks,
                                     self.rlk, 3, self.keys[0], 3, self.keys[1], scores=self.scores,
                                     context=self.context, sum_before_scaling=True)

    def clear(self):
        for t in (self.scores, self.context, self.cache.view(6, 2, -1)[:, 1]):
            t.zero_()

    def results(self):
        return [t.clone() for t in (self.scores, self.context, self.cache)]

    def matches(self, want):
        return all(self.torch.equal(a, b) for a, b in zip(self.results(), want))


def _alone(step):
    step()
    step.torch.cuda.synchronize()
    return step.results()


def test_two_threads_step_two_contexts_on_two_streams():
    import torch
    steps = [Step("C1", 1), Step("C2", 2)]
    want = [_alone(s) for s in steps]
    for s in steps:
        s.clear()
    torch.cuda.synchronize()
    say("two threads, twenty steps each")
    failed = []

    def work(step):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(20):
                    step()
            stream.synchronize()
        except Exception as e:       # reported by the assertion below
            failed.append(e)

    threads = [threading.Thread(target=work, args=(s,)) for s in steps]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    for s, w in zip(steps, want):
        assert s.matches(w)


def test_a_captured_step_replays_beside_steps_of_another_context():
    import torch
    step, other = Step("C1", 3), Step("C2", 4)
    want, want_other = _alone(step), _alone(other)
    say("capture with a second context alive")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    torch.cuda.synchronize()
    for rep in range(3):
        say(f"replay {rep}")
        step.clear()
        other.clear()
        torch.cuda.synchronize()
        other()                          # eager, on the default stream
        with torch.cuda.stream(side):
            graph.replay()
        other()
        torch.cuda.synchronize()
        assert step.matches(want), rep
        assert other.matches(want_other), rep
        step()                           # eager steps of the captured context between replays
        torch.cuda.synchronize()
        assert step.matches(want), rep
