"""Replays of every form of captured graph: one launch of the library (replayed
as that launch), a few (replayed as launches where the HIP runtime does not keep
a graph together either), many, and launches mixed with another library's kernel
or made on a second stream (replayed as a graph).  Every replay, with changed inputs
and other work between, equals the eager result, and is one operation to other
threads' calls on its stream."""
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

try:
    import torch

    import paper_2609_37532_amd as dsv
    from gpu_util import DEV, AcceptDev, DvlDev
except Exception:  # pragma: no cover
    pass


def inputs(seed):
    rng = np.random.default_rng(seed)
    qlens = [5, 16, 1, 9]
    return W.make_accept_inputs(rng, cu_qlens=W.cu_from_lengths(qlens), capacity=34, vocab=9001,
                                dtype="bf16")


def few(launches):
    """What direct_launches() is for a few launches of the library alone."""
    major, minor = (int(x) for x in torch.version.hip.split(".")[:2])
    return launches if (major, minor) < (7, 1) else 0


@pytest.mark.parametrize("calls,foreign", [(1, False), (3, False), (4, False), (8, False),
                                           (9, False), (2, True)])
def test_replays_equal_eager(calls, foreign):
    # calls of accept are two launches each
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
    assert g.direct_launches() == (few(2 * calls) if calls <= 3 and not foreign else 0)
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


def dvl_inputs(seed):
    return W.make_dvl_inputs(np.random.default_rng(seed), n_bs=70, n_live=61 - seed % 7)


def dvl_result(d):
    return np.concatenate([v.view(np.int32).ravel() for v in d.result().values()])


@pytest.mark.parametrize("form", ["one", "two", "foreign", "side stream", "both streams"])
def test_what_is_replayed_as_launches(form):
    d = DvlDev(dvl_inputs(0))
    stream, side, third = (torch.cuda.Stream() for _ in range(3))
    count = torch.zeros(1, dtype=torch.int32, device=DEV)

    def work():
        if "stream" in form:  # forked off the captured stream, and joined again
            side.wait_stream(stream)
            d.run(stream=side)
            stream.wait_stream(side)
        if form != "side stream":
            d.run(stream=stream)
        if form == "two":
            d.run(stream=stream)
        if form == "foreign":
            with torch.cuda.stream(stream):
                count.add_(1)

    work()
    torch.cuda.synchronize()
    g = dsv.Graph().capture(work, stream)
    assert g.direct_launches() == {"one": 1, "two": few(2)}.get(form, 0)
    null = torch.cuda.default_stream()
    for step, on in enumerate([stream, third, "captured", null, stream]):
        new = DvlDev(dvl_inputs(1 + step))
        new.run()
        for name in ("logits", "num_live", "tokens", "positions", "kv_refs"):
            getattr(d, name).copy_(getattr(new, name))
        for out in (d.k, d.cu, d.ptok, d.ppos, d.pref, d.scores):
            out.fill_(DvlDev.POISON)
        torch.cuda.synchronize()
        if on == "captured":
            # into a stream that is being captured: run at once or with the
            # graph that is captured, as the runtime has it, but always run
            outer = dsv.Graph().capture(lambda: g.replay(third), third)
            assert outer.direct_launches() == 0
            outer.replay(third)
        else:
            g.replay(on)
        assert np.array_equal(dvl_result(d), dvl_result(new)), (form, step)
    g.close()


def beside(work):
    """Runs work(stopped) in a thread; leaving the context ends and joins it."""
    class Beside:
        def __enter__(self):
            self.stop = threading.Event()
            self.error = None
            self.thread = threading.Thread(target=self.run)
            self.thread.start()

        def run(self):
            try:
                work(self.stop.is_set)
            except Exception as e:  # reported by the test's thread
                self.error = e

        def __exit__(self, *exc):
            self.stop.set()
            self.thread.join()
            assert self.error is None, self.error
            return False

    return Beside()


@pytest.mark.parametrize("calls", [1, 6, 18])
def test_no_call_of_another_thread_comes_inside_a_replay(calls):
    # calls that read one input, which another thread's calls overwrite on the
    # same stream: within a replay all of them saw the same value
    n_bs, w = 8, 16
    d = DvlDev(W.make_dvl_inputs(np.random.default_rng(3), n_bs=n_bs, n_live=n_bs))
    ones = [torch.full_like(d.tokens, v) for v in (1, 2)]
    half = d.tokens.view(-1)[:w * n_bs // 2]  # written by the other thread's packing
    stream, steps = torch.cuda.Stream(), 400
    outs = lambda: [torch.zeros_like(x) for x in (d.k, d.cu, d.ppos, d.pref)]  # noqa: E731
    mine, theirs = outs(), outs()
    packed = torch.zeros((calls, d.ptok.numel()), dtype=torch.int32, device=DEV)
    seen = torch.zeros((steps, *packed.shape), dtype=torch.int32, device=DEV)

    def pack(tokens, into, o):
        dsv.dvl_allocate_pack(d.logits, d.num_live, tokens, d.positions, d.kv_refs, o[0], o[1],
                              into, o[2], o[3], stream=stream)

    started = threading.Event()

    def overwrite(stopped):
        for n in range(100_000):
            if stopped():
                break
            pack(ones[n % 2], half, theirs)
            started.set()

    d.tokens.fill_(1)
    torch.cuda.synchronize()
    g = dsv.Graph().capture(lambda: [pack(d.tokens, out, mine) for out in packed], stream)
    assert g.direct_launches() == {1: 1, 6: few(6), 18: 0}[calls]
    with beside(overwrite):
        started.wait(30)
        for step in range(steps):
            g.replay(stream)
            with torch.cuda.stream(stream):
                seen[step].copy_(packed)
    torch.cuda.synchronize()
    g.close()
    rows = seen.cpu().numpy()
    assert np.unique(rows[:, 0, 0]).size == 2  # the other thread's calls were there
    torn = [step for step in range(steps) if (rows[step] != rows[step, 0]).any()]
    assert not torn, (len(torn), rows[torn[0]][:, 0])


def test_two_threads_replay_graphs_that_share_a_stream_and_a_workspace():
    x, y = AcceptDev(inputs(11)), AcceptDev(inputs(12))
    y.ws = x.ws
    want = []
    for d in (x, y):
        d.run()
        want.append(np.stack(d.result()))
    assert not np.array_equal(want[0], want[1])
    stream = torch.cuda.Stream()
    graphs = [dsv.Graph().capture(lambda d=d: d.run(stream=stream), stream) for d in (x, y)]
    steps = 300
    seen = torch.zeros((2, steps, 2, want[0].shape[1]), dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()

    def replays(n, d):
        for step in range(steps):
            graphs[n].replay(stream)
            with torch.cuda.stream(stream):
                seen[n, step, 0].copy_(d.a)
                seen[n, step, 1].copy_(d.nxt)

    with beside(lambda stopped: replays(1, y)):
        replays(0, x)
    torch.cuda.synchronize()
    got = seen.cpu().numpy()
    for n in range(2):
        assert (got[n] == want[n][None]).all(), n
        graphs[n].close()
