"""The Fourier measurement's kernels at the edges of their forms: a replica in
one chunk and in several, rows of whole dwords and others, bit for bit against
the sums written out here (the C oracle's compiler joins its cos and sin calls
into one sincos, whose last bit differs at L = 40); in a batch and in a pool whose membership and measurement flags
change, against single runs."""
import math

import numpy as np
import pytest

from paper_1508_06268_amd import workloads as W
from parity_util import make_pair

pytestmark = pytest.mark.gpu


def _sample(s, L):
    """F of one configuration: plane sums, then FP64 with v ascending."""
    a = s.reshape(L, L, L).astype(np.int64)
    total = 0.0
    for n in (a.sum((0, 1)), a.sum((0, 2)), a.sum((1, 2))):
        c = q = 0.0
        for v in range(L):
            x = 2.0 * math.pi * float(v) / float(L)
            c += math.cos(x) * float(n[v])
            q += math.sin(x) * float(n[v])
        total += c * c
        total += q * q
    return total / (3.0 * float(L ** 3))


@pytest.mark.parametrize("L,R", [(2, 2), (6, 3), (8, 5), (10, 2), (24, 3), (32, 4), (36, 2), (40, 2), (48, 2), (64, 3), (128, 1)])
def test_samples_match_the_written_sums(rfim_mod, oracle_mod, L, R):
    f = W.bimodal_fields(L, [71, L])
    T = W.linear_temps(R, 3.0, 5.0) if R > 1 else np.array([4.0])
    g, o = make_pair(rfim_mod, oracle_mod, L, R, 1.0, 1.0, f, T, seed=L)
    g.set_measure(rfim_mod.MEASURE_FOURIER)
    want = np.zeros((R, 2))
    for _ in range(2):
        g.sweep(2, 2)
        o.sweep(2, 2)
        spins, perm = o.spins(), o.perm()
        want[:, 0] += 1
        want[:, 1] += [_sample(spins[perm[t]], L) for t in range(R)]
    assert np.array_equal(g.fourier(), want)
    g.close()
    o.close()


def _spec(L, R, q):
    return W.Realization(L=L, R=R, J=1.0, h=1.0, fields=W.bimodal_fields(L, [72, L, q]), temps=W.linear_temps(R, 3.0, 5.0),
                         seed=5, realization=q, sweeps=0, every=2)


def _single(rfim_mod, w, before, after):
    g = rfim_mod.Rfim(w.L, w.R, w.J, w.h, w.fields, w.temps, seed=w.seed, realization=w.realization)
    if before:
        g.sweep(before, 2)
    g.set_measure(rfim_mod.MEASURE_FOURIER)
    g.sweep(after, 2)
    out = g.fourier()
    g.close()
    return out


def test_batch_of_all_chunk_counts(rfim_mod):
    specs = [_spec(8, 3, 0), _spec(64, 2, 1), _spec(32, 2, 2), _spec(64, 3, 3), _spec(16, 4, 4)]
    b = rfim_mod.Batch(specs)
    b.set_shape(64, 0, 0, 4, 128)
    for q in (0, 1, 2, 4):
        b.item(q).set_measure(rfim_mod.MEASURE_FOURIER)
    b.sweep(8, 2)
    for q in (0, 1, 2, 4):
        assert np.array_equal(b.item(q).fourier(), _single(rfim_mod, specs[q], 0, 8)), q
    assert not b.item(3).fourier().any()
    b.item(3).set_measure(rfim_mod.MEASURE_FOURIER)
    b.item(1).set_measure(0)
    held = b.item(1).fourier()
    b.sweep(4, 2)
    assert np.array_equal(b.item(3).fourier(), _single(rfim_mod, specs[3], 8, 4))
    assert np.array_equal(b.item(1).fourier(), held)
    b.close()


def test_pool_items_measured_across_membership_changes(rfim_mod):
    specs = [_spec(16, 4, 6), _spec(32, 3, 7), _spec(8, 5, 8)]
    p = rfim_mod.Pool(1 << 30)
    a = p.admit(specs[0])
    p.step(4, 2)
    p.item(a).set_measure(rfim_mod.MEASURE_FOURIER)
    c = p.admit(specs[1])
    p.item(c).set_measure(rfim_mod.MEASURE_FOURIER)
    p.step(4, 2)
    d = p.admit(specs[2])
    p.step(2, 2)
    assert np.array_equal(p.item(a).fourier(), _single(rfim_mod, specs[0], 4, 6))
    assert np.array_equal(p.item(c).fourier(), _single(rfim_mod, specs[1], 0, 6))
    assert not p.item(d).fourier().any()
    p.release(a)
    p.step(2, 2)
    assert np.array_equal(p.item(c).fourier(), _single(rfim_mod, specs[1], 0, 8))
    p.close()


def test_captured_step_does_not_depend_on_later_flags(rfim_mod):
    """A pool step captured right after an item's measurement was turned on,
    and replayed after another item's was, whose steps lay the launches of the
    whole pool out anew: the recorded items are measured, at each replay."""
    import torch

    specs = [_spec(16, 4, 9), _spec(32, 3, 10), _spec(64, 2, 11)]
    stream = torch.cuda.Stream()
    p = rfim_mod.Pool(1 << 30, stream=stream)
    p.set_shape(64, rfim_mod.FIELDS_BIMODAL, 0, 4, 128)
    ids = [p.admit(w) for w in specs]
    p.step(4, 2)
    for q in (0, 2):
        p.item(ids[q]).set_measure(rfim_mod.MEASURE_FOURIER)
    p.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
        p.step(2, 2)
    with torch.cuda.stream(stream):         # the replays in order with the pool's own work
        graph.replay()
        p.item(ids[1]).set_measure(rfim_mod.MEASURE_FOURIER)
        p.step(4, 2)
        graph.replay()
        graph.replay()
    for q, before, after in ((0, 4, 10), (1, 6, 4), (2, 4, 10)):
        assert np.array_equal(p.item(ids[q]).fourier(), _single(rfim_mod, specs[q], before, after)), q
    p.close()
