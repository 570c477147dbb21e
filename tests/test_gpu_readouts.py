"""Readouts of a handle: counters, permutations, energies and configurations
through pinned memory, at the sizes where their launches change form (a
workgroup per replica, several per replica, rows of 16 sites or fewer, pieces
of a configuration) and behind work that takes longer than their polling."""
import numpy as np
import pytest

from helpers import energy_numpy
from paper_1508_06268_amd import workloads as W

pytestmark = pytest.mark.gpu


def check_state(g, f, L, R, h):
    s, perm = g.spins(), g.perm()
    E, M = g.energies(), g.magnetizations()
    assert sorted(perm) == list(range(R))
    for slot in (0, R // 2, R - 1):
        r = int(perm[slot])
        want, _ = energy_numpy(s[r], f, L, 1.0, h)
        assert M[slot] == s[r].sum()
        assert np.isclose(E[slot], want, rtol=1e-12, atol=1e-9)     # FP64 sums of N terms in another order


@pytest.mark.parametrize("L,R", [(2, 1), (6, 3), (8, 300), (22, 9), (24, 9), (30, 5), (32, 40), (34, 5), (64, 20)])
@pytest.mark.parametrize("kind", ["b", "g"])
def test_readouts_behind_queued_work(rfim_mod, L, R, kind):
    """Every call reads the state after all sweeps queued before it, whether
    the wait for it is short or long, and twice the same."""
    f = W.bimodal_fields(L, [91, L]) if kind == "b" else W.gaussian_fields(L, [91, L])
    T = W.linear_temps(R, 1.5, 4.0) if R > 1 else np.array([2.0])
    g = rfim_mod.Rfim(L, R, 1.0, 1.5, f, T, seed=3)
    for n in (1, 400):
        g.sweep(n, 1)
        E = g.energies()
        att = np.asarray(g.exchange_stats()[0]) if R > 1 else None
        assert np.array_equal(E, g.energies())
        check_state(g, f, L, R, 1.5)
        if R > 1:
            k = n if n == 1 else 401
            assert list(att) == [(k + 1 - (p & 1)) // 2 for p in range(R - 1)]
    g.close()


@pytest.mark.parametrize("L,R", [(2, 3), (6, 2), (16, 5), (20, 700), (32, 130), (64, 17), (128, 3)])
def test_configurations_round_trip(rfim_mod, L, R):
    """set_spins then spins: every layout, and more than one piece of 4 MiB
    (L = 20, R = 700; L = 64, R = 17 and L = 128, R = 3 in bits); and what
    was there stays when one value is not +-1."""
    rng = np.random.default_rng([92, L])
    f = W.bimodal_fields(L, [92, L])
    g = rfim_mod.Rfim(L, R, 1.0, 1.5, f, W.linear_temps(R, 1.5, 4.0), seed=3)
    s = (2 * rng.integers(0, 2, size=(R, L ** 3)) - 1).astype(np.int8)
    g.set_spins(s)
    assert np.array_equal(np.asarray(g.spins()).reshape(R, -1), s)
    check_state(g, f, L, R, 1.5)
    bad = s.copy()
    bad[R - 1, L ** 3 - 1] = 0
    with pytest.raises(rfim_mod.RfimError):
        g.set_spins(bad)
    assert np.array_equal(np.asarray(g.spins()).reshape(R, -1), s)
    g2 = rfim_mod.Rfim.load(g.save())
    assert np.array_equal(np.asarray(g2.spins()).reshape(R, -1), s)
    g.close()
    g2.close()


@pytest.mark.parametrize("R", [1, 2, 3, 5, 170, 171, 255, 1023, 1024, 1025, 2731, 4099, 5000])
def test_arrays_of_every_length(rfim_mod, R):
    """Permutations (R words), counters and per-slot sums (2 to 12 words a
    replica): lengths around a workgroup's share, of several steps and with
    one to three words at the end."""
    f = W.bimodal_fields(2, [95])
    g = rfim_mod.Rfim(2, R, 1.0, 1.5, f, W.linear_temps(R, 1.5, 4.0) if R > 1 else np.array([2.0]), seed=3)
    p = np.random.default_rng(R).permutation(R).astype(np.int32)
    g.set_perm(p)
    assert np.array_equal(g.perm(), p)
    g.sweep(1, 1)
    E, M, obs = g.energies(), g.magnetizations(), g.observables()
    want = np.stack([np.ones(R), E, E * E, np.abs(M), 1.0 * M * M, 1.0 * M ** 4], axis=1)
    assert np.array_equal(obs, want)
    att, acc = g.exchange_stats()
    assert np.array_equal(att, (np.arange(R - 1) + 1) % 2) and np.all(acc <= att)
    assert sorted(g.perm()) == list(range(R)) and (g.perm() != p).sum() == 2 * acc.sum()
    assert g.counters() == (1, 1)
    g.close()


def test_readouts_that_fail_leave_later_ones_alone(rfim_mod):
    """A readout behind 20 ms of sweeps, in a thread that captures another
    stream: its wait is refused and the call fails.  When its kernels end, they
    write into no other call's results."""
    import ctypes
    import time

    import torch

    hip = ctypes.CDLL("libamdhip64.so")
    L, R = 16, 32
    f = W.bimodal_fields(L, [94, L])
    far, near = (rfim_mod.Rfim(L, R, 1.0, 1.5, f, W.linear_temps(R, 1.5, 4.0), seed=q) for q in (1, 2))
    near.sweep(5, 1)
    E = near.energies()
    far.sweep(1, 1)
    far.synchronize()
    t = time.perf_counter()
    far.sweep(1000, 0)
    far.synchronize()
    n = int(20e-3 / (time.perf_counter() - t) * 1000)
    other = torch.cuda.Stream()
    for _ in range(12):
        torch.cuda.synchronize()
        far.sweep(n, 0)
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(other.cuda_stream), 1) == 0
        failed = False
        try:
            far.energies()
        except rfim_mod.RfimError:
            failed = True
        graph = ctypes.c_void_p()
        hip.hipStreamEndCapture(ctypes.c_void_p(other.cuda_stream), ctypes.byref(graph))
        hip.hipGetLastError()
        until = time.perf_counter() + 30e-3
        while failed and time.perf_counter() < until:
            assert np.array_equal(near.energies(), E)
    far.synchronize()
    check_state(far, f, L, R, 1.5)
    far.close()
    near.close()
