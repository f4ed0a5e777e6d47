"""Replays of every form of captured graph: a few launches of the library
(replayed as launches), many of them, and launches mixed with another
library's kernel (replayed as a graph).  Every replay, with changed inputs and
other work between, equals the eager result."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

try:
    import torch

    import paper_2609_37532_amd as dsv
    from gpu_util import DEV, AcceptDev
except Exception:  # pragma: no cover
    pass


def inputs(seed):
    rng = np.random.default_rng(seed)
    qlens = [5, 16, 1, 9]
    return W.make_accept_inputs(rng, cu_qlens=W.cu_from_lengths(qlens), capacity=34, vocab=9001,
                                dtype="bf16")


@pytest.mark.parametrize("calls,foreign", [(1, False), (8, False), (9, False), (2, True)])
def test_replays_equal_eager(calls, foreign):
    # calls of accept are two launches each: 2, 16 and 18 launches
    d, other = AcceptDev(inputs(calls)), AcceptDev(inputs(100 + calls))
    stream = torch.cuda.Stream()
    count = torch.zeros(1, dtype=torch.int32, device=DEV)

    def work():
        for _ in range(calls):
            d.run(stream=stream)
            if foreign:
                with torch.cuda.stream(stream):
                    count.add_(1)

    work()
    torch.cuda.synchronize()
    count.zero_()
    g = dsv.Graph().capture(work, stream)
    torch.cuda.synchronize()
    assert int(count) == 0  # captured, not run
    for step in range(4):
        new = AcceptDev(inputs(1000 * calls + step))
        new.run()
        for dst, src in ((d.logits, new.logits), (d.draft, new.draft)):
            dst.copy_(src)
        d.a.fill_(-7)
        d.nxt.fill_(-7)
        other.run()
        torch.cuda.synchronize()
        g.replay(stream)
        a, nxt = d.result()
        ra, rn = new.result()
        assert np.array_equal(a, ra) and np.array_equal(nxt, rn), step
        if foreign:
            assert int(count) == calls * (step + 1)
    g.close()


def test_replay_on_another_stream_and_two_captures_at_once():
    # two streams captured by one thread at the same time, replayed on a third
    x, y = AcceptDev(inputs(1)), AcceptDev(inputs(2))
    s1, s2, s3 = (torch.cuda.Stream() for _ in range(3))
    for d in (x, y):
        d.run()
    want = [x.result(), y.result()]
    g2 = dsv.Graph()
    g1 = dsv.Graph().capture(
        lambda: (x.run(stream=s1), g2.capture(lambda: y.run(stream=s2), s2)), s1)
    for d in (x, y):
        d.a.fill_(-7)
        d.nxt.fill_(-7)
    torch.cuda.synchronize()
    g1.replay(s3)
    g2.replay(s3)
    for d, (a, n) in zip((x, y), want):
        ga, gn = d.result()
        assert np.array_equal(ga, a) and np.array_equal(gn, n)
    g1.close()
    g2.close()
