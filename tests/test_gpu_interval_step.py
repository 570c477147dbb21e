"""Calls of several exchange intervals on shapes whose launches run whole
intervals: the step between two intervals runs inside the first launch of the
next one, the last one by itself.  +-1 fields follow the oracle bit for bit;
with continuous fields one call ends in the state of single intervals, whose
steps are all of the second kind."""
import numpy as np
import pytest

from paper_1508_06268_amd import workloads as W
from parity_util import assert_same_state, make_pair

pytestmark = pytest.mark.gpu

# (L, R, launch shape or None for the default): resident; slabs of one, two and
# three sweeps a launch; boxes and residents of other sizes; around the largest
# ladder (R times the partials per replica up to 256) that takes the step so
SHAPES = [(8, 1, None), (8, 2, None), (8, 5, None), (8, 256, None), (8, 257, None), (16, 7, None), (16, 6, (2, 4, 256)),
          (32, 3, (1, 4, 1024)), (32, 5, (2, 8, 512)), (32, 64, (3, 4, 1024)), (32, 3, (4, 2, 1024)), (22, 3, None),
          (24, 9, None), (24, 60, None), (40, 3, None), (48, 5, None), (6, 300, None)]


def ladder(R, L):
    return W.linear_temps(R, 2.0, 2.0 + 0.002 * (R - 1) * (64 / L) ** 1.5) if R > 1 else np.array([2.0])


@pytest.mark.parametrize("L,R,shape", SHAPES)
def test_intervals_match_oracle(rfim_mod, oracle_mod, L, R, shape):
    f = W.bimodal_fields(L, [101, L])
    g, o = make_pair(rfim_mod, oracle_mod, L, R, 1.0, 1.5, f, ladder(R, L), seed=L, realization=R)
    if shape:
        g.set_launch_shape(*shape)
    for n, every in ((9, 3), (4, 4), (7, 2), (5, 0), (3, 1)):     # ends on a step, one step, ends off one, none, each sweep
        g.sweep(n, every)
        o.sweep(n, every)
        assert_same_state(g, o, "L=%d R=%d (%d, %d)" % (L, R, n, every))
    g.close()
    o.close()


@pytest.mark.parametrize("L,R,shape", SHAPES)
def test_one_call_equals_single_intervals(rfim_mod, L, R, shape):
    f = W.gaussian_fields(L, [102, L])
    out = []
    for calls in ([(15, 3), (4, 3)], [(3, 3)] * 5 + [(4, 3)]):
        g = rfim_mod.Rfim(L, R, 1.0, 1.5, f, ladder(R, L), seed=L, realization=R)
        if shape:
            g.set_launch_shape(*shape)
        for n, every in calls:
            g.sweep(n, every)
        att, acc = g.exchange_stats()
        out.append((g.spins(), g.perm(), g.observables(), att, acc, g.energies()))
        g.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("L,R", [(8, 16), (32, 6), (24, 5)])
def test_two_handles_on_one_stream_and_two_threads(rfim_mod, L, R):
    """The pending steps' state is the call's own: handles that take turns on
    one stream, and handles of two threads, end as each does alone."""
    import threading

    import torch

    def make(q, stream=None):
        f = W.bimodal_fields(L, [103, L, q])
        return rfim_mod.Rfim(L, R, 1.0, 1.5, f, ladder(R, L), seed=q, stream=stream)

    def state(g):
        return g.spins(), g.perm(), g.observables(), g.energies()

    alone = []
    for q in range(2):
        g = make(q)
        g.sweep(40, 4)
        g.sweep(20, 4)
        alone.append(state(g))
        g.close()
    stream = torch.cuda.Stream()
    pair = [make(q, stream) for q in range(2)]
    for n in (40, 20):
        for g in pair:
            g.sweep(n, 4)
    got = [state(g) for g in pair]
    for g in pair:
        g.close()
    threaded = [None, None]

    def work(q):
        g = make(q)
        g.sweep(40, 4)
        g.sweep(20, 4)
        threaded[q] = state(g)
        g.close()

    ts = [threading.Thread(target=work, args=(q,)) for q in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for q in range(2):
        for a, b, c in zip(alone[q], got[q], threaded[q]):
            assert np.array_equal(a, b) and np.array_equal(a, c)


@pytest.mark.parametrize("L,R", [(8, 5), (16, 3), (22, 4), (32, 3), (40, 3), (48, 30), (60, 2)])
def test_captured_call_goes_on_at_each_replay(rfim_mod, oracle_mod, L, R):
    """A call captured on the handle's stream: every replay runs the next
    sweeps and steps, as the next call would."""
    import torch

    f = W.bimodal_fields(L, [104, L])
    stream = torch.cuda.Stream()
    g = rfim_mod.Rfim(L, R, 1.0, 1.5, f, ladder(R, L), seed=L, stream=stream)
    o = oracle_mod.Oracle(L, R, 1.0, 1.5, f, ladder(R, L), seed=L)
    g.sweep(4, 2)
    o.sweep(4, 2)
    g.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        g.sweep(6, 2)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        o.sweep(6, 2)
        assert np.array_equal(g.spins(), o.spins()) and np.array_equal(g.perm(), o.perm())
        assert np.array_equal(g.energies(), o.energies())
    for a, b in zip(g.exchange_stats(), o.exchange_stats()):
        assert np.array_equal(a, b)
    g.close()
    o.close()


@pytest.mark.parametrize("kind", ["b", "g"])
@pytest.mark.parametrize("L,R,bimodal,gaussian", [
    (16, 256, (1, 1, 512), (1, 1, 512)), (16, 257, (1, 2, 256), (1, 2, 256)),
    (32, 32, (4, 8, 1024), (4, 8, 1024)), (32, 33, (1, 4, 1024), (3, 4, 1024)),
    (32, 65, (1, 4, 1024), (1, 4, 1024))])
def test_default_shapes(rfim_mod, L, R, bimodal, gaussian, kind):
    """The shape a handle starts on follows its capacity; the chain does not."""
    f = W.bimodal_fields(L, [105, L]) if kind == "b" else W.gaussian_fields(L, [105, L])
    out = []
    for cap, shape in ((R, None), (R, (1, 2, 256)), (R + 300, None)):
        g = rfim_mod.Rfim(L, R, 1.0, 1.5, f, ladder(R, L), seed=L, R_cap=cap)
        if shape:
            g.set_launch_shape(*shape)
        elif cap == R:
            assert g.launch_shape() == (bimodal if kind == "b" else gaussian)
        else:
            assert g.launch_shape() == ((1, 2, 256) if L == 16 else (1, 4, 1024))
        g.sweep(11, 5)
        out.append((g.spins(), g.perm()))
        g.close()
    for other in out[1:]:
        assert np.array_equal(out[0][0], other[0]) and np.array_equal(out[0][1], other[1])


@pytest.mark.parametrize("R", [1, 3, 512, 513])
@pytest.mark.parametrize("hot", [True, False])
def test_l8_intervals_of_every_length(rfim_mod, oracle_mod, R, hot):
    """L = 8 around the batches of random words (12 sweeps) and the largest
    ladder that uses them; cold: temperatures at which classes never flip."""
    f = W.bimodal_fields(8, [106, R])
    T = ladder(R, 8) if hot else np.linspace(0.03, 0.6, R)
    g, o = make_pair(rfim_mod, oracle_mod, 8, R, 1.0, 1.5, f, T, seed=7)
    for n, every in ((12, 12), (13, 13), (50, 25), (24, 24), (31, 0), (2, 1)):
        g.sweep(n, every)
        o.sweep(n, every)
        assert_same_state(g, o, "R=%d (%d, %d)" % (R, n, every))
    g.close()
    o.close()


@pytest.mark.parametrize("R", [2, 512])
def test_l8_continuous_fields_do_not_depend_on_the_shape(rfim_mod, R):
    f = W.gaussian_fields(8, [107, R])
    out = []
    for shape in (None, (1, 1, 128)):
        g = rfim_mod.Rfim(8, R, 1.0, 1.5, f, ladder(R, 8), seed=9)
        if shape:
            g.set_launch_shape(*shape)
        for n, every in ((12, 12), (13, 13), (50, 25), (31, 0)):
            g.sweep(n, every)
        out.append((g.spins(), g.perm()))
        g.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("seed", [1, 2])
def test_second_streams_among_batches(rfim_mod, seed):
    """Two-stream handles on their own and on torch's streams, between batches
    that come and go (whose creation drops the idle second streams): each ends
    as it does on one stream."""
    import torch

    rng = np.random.default_rng([108, seed])
    f = W.bimodal_fields(64, [108, 64])
    T = W.linear_temps(8, 1.5, 4.0)
    one = rfim_mod.Rfim(64, 8, 1.0, 1.5, f, T, seed=3)
    one.set_concurrency(1)
    one.sweep(12, 4)
    want = one.spins(), one.perm(), one.energies()
    kept = []
    for q in range(8):
        if rng.random() < 0.5:
            specs = [W.Realization(L=L, R=4, J=1.0, h=1.0, fields=W.bimodal_fields(L, [109, L]), temps=W.linear_temps(4, 1.5, 4.0),
                                   seed=1, realization=L, every=2) for L in (8, 16, 32)]
            b = rfim_mod.Batch(specs)
            b.sweep(4, 2)
            b.synchronize()
            b.close()
        g = rfim_mod.Rfim(64, 8, 1.0, 1.5, f, T, seed=3, stream=torch.cuda.Stream() if rng.random() < 0.5 else None)
        g.set_concurrency(2)
        g.sweep(12, 4)
        for a, b in zip((g.spins(), g.perm(), g.energies()), want):
            assert np.array_equal(a, b)
        kept.append(g)
        if len(kept) > 3:
            kept.pop(0).close()
    for g in kept + [one]:
        g.close()


@pytest.mark.parametrize("L,R", [(8, 5), (32, 3), (40, 3)])
def test_exchange_counter_beyond_32_bits(rfim_mod, oracle_mod, L, R):
    """From the largest counter that can be set: the random words take its low
    half, the counter itself goes on."""
    f = W.bimodal_fields(L, [116, L])
    g, o = make_pair(rfim_mod, oracle_mod, L, R, 1.0, 1.5, f, ladder(R, L), seed=L)
    for h in (g, o):
        h.set_counters(7, 2 ** 32 - 1)
    for n, every in ((9, 2), (4, 4), (3, 1)):
        g.sweep(n, every)
        o.sweep(n, every)
        assert_same_state(g, o, "(%d, %d)" % (n, every))
    g.close()
    o.close()


def captured_between_ordinary_calls(rfim_mod, ref, L, R, f, shape=None):
    """A captured call, replayed before, between and after ordinary calls of
    one launch an interval and of an odd number of them: all of them are one
    chain, the one that ref runs in ordinary calls alone."""
    import torch

    stream = torch.cuda.Stream()
    g = rfim_mod.Rfim(L, R, 1.0, 1.5, f, ladder(R, L), seed=L, stream=stream)
    if shape:
        g.set_launch_shape(*shape)
    g.sweep(4, 2)
    ref.sweep(4, 2)
    g.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        g.sweep(6, 2)
    for what in ("replay", "replay", (6, 2), "replay", (3, 1), (5, 0), "replay", "replay", (4, 4), (2, 1), "replay"):
        if what == "replay":
            graph.replay()
            torch.cuda.synchronize()
            ref.sweep(6, 2)
        else:
            g.sweep(*what)
            ref.sweep(*what)
        assert np.array_equal(g.spins(), ref.spins()) and np.array_equal(g.perm(), ref.perm()), what
        assert np.array_equal(g.energies(), ref.energies()), what
    for a, b in zip(g.exchange_stats(), ref.exchange_stats()):
        assert np.array_equal(a, b)
    g.close()
    ref.close()


@pytest.mark.parametrize("L,R", [(8, 5), (16, 3), (22, 4), (12, 40)])
def test_ordinary_calls_between_replays_in_place(rfim_mod, oracle_mod, L, R):
    f = W.bimodal_fields(L, [110, L])
    captured_between_ordinary_calls(rfim_mod, oracle_mod.Oracle(L, R, 1.0, 1.5, f, ladder(R, L), seed=L), L, R, f)


@pytest.mark.parametrize("kind", ["b", "g"])
@pytest.mark.parametrize("L,R", [(16, 3), (32, 3), (24, 3), (28, 2), (40, 3), (48, 30)])
def test_ordinary_calls_between_replays_two_buffers(rfim_mod, oracle_mod, L, R, kind):
    """Slabs and boxes, whose ordinary launches go from one spin buffer to the
    other (L = 16: slabs set by hand; +-1 fields against the oracle, continuous
    ones against a handle without a captured call)."""
    if kind == "b":
        f = W.bimodal_fields(L, [111, L])
        ref = oracle_mod.Oracle(L, R, 1.0, 1.5, f, ladder(R, L), seed=L)
    else:
        f = W.gaussian_fields(L, [111, L])
        ref = rfim_mod.Rfim(L, R, 1.0, 1.5, f, ladder(R, L), seed=L)
    captured_between_ordinary_calls(rfim_mod, ref, L, R, f, (2, 2, 512) if L == 16 else None)


def us_a_sweep(g, n=50):
    import time

    out = []
    for _ in range(9):
        t = time.perf_counter()
        g.sweep(n, 10)
        g.synchronize()
        out.append((time.perf_counter() - t) / n * 1e6)
    return min(out)


@pytest.mark.parametrize("gone", [(2,), (0, 2), (1, 3)])
def test_two_stream_handles_stay_side_by_side(rfim_mod, gone):
    """Handles that stay while others and a batch come and go sweep as fast as
    before: on a pair of streams that takes turns a sweep takes 3.5 times as
    long (bound: twice)."""
    import torch

    f, T = W.bimodal_fields(64, [112]), W.linear_temps(128, 1.0, 6.0)
    hs = []
    for q in range(6):
        hs.append(rfim_mod.Rfim(64, 128, 1.0, 1.5, f, T, seed=q, stream=torch.cuda.Stream() if q % 2 else None))
        hs[-1].sweep(10, 10)
    before = [us_a_sweep(g) for g in hs]
    for q in gone:
        hs[q].close()
    specs = [W.Realization(L=L, R=4, J=1.0, h=1.0, fields=W.gaussian_fields(L, [113, L]), temps=W.linear_temps(4, 1.5, 4.0),
                           seed=1, realization=L, every=10) for L in (8, 16, 32)]
    b = rfim_mod.Batch(specs)
    b.sweep(40, 10)
    b.synchronize()
    kept = [q for q in range(6) if q not in gone]
    assert all(us_a_sweep(hs[q]) < 2.0 * before[q] for q in kept), (before, [us_a_sweep(hs[q]) for q in kept])
    b.close()
    for q in kept:
        hs[q].close()


def test_batches_between_large_handles_cost_no_new_stream(rfim_mod):
    """A loop of a two-stream handle and a batch: from the second turn on the
    handle's first call takes no longer than the next one and what a trial of
    its streams takes (0.2 ms; setting up a hardware queue takes 4)."""
    import time

    f, T = W.bimodal_fields(64, [114]), W.linear_temps(128, 1.0, 6.0)
    specs = [W.Realization(L=L, R=4, J=1.0, h=1.0, fields=W.gaussian_fields(L, [115, L]), temps=W.linear_temps(4, 1.5, 4.0),
                           seed=1, realization=L, every=10) for L in (8, 16, 32)]
    extra = []
    for _ in range(9):
        g = rfim_mod.Rfim(64, 128, 1.0, 1.5, f, T, seed=3)
        g.synchronize()
        took = []
        for _ in range(2):
            t = time.perf_counter()
            g.sweep(20, 10)
            g.synchronize()
            took.append((time.perf_counter() - t) * 1e3)
        extra.append(took[0] - took[1])
        g.close()
        b = rfim_mod.Batch(specs)
        b.sweep(40, 10)
        b.synchronize()
        b.close()
    assert np.median(extra[2:]) < 2.0, extra
