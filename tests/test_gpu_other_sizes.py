"""Lattice sizes that are not powers of two (and L = 2, 4): the LDS-resident
form, boxes (slabs and whole replicas), the streaming half-sweeps, rows of
whole dwords and rows that end inside one.  +-1 fields follow the oracle bit for bit; of one sweep's decisions with
continuous fields at most one differs (they are FP32 on the device: about 1 in
3e7)."""
import numpy as np
import pytest

from helpers import energy_numpy, quench_numpy
from paper_1508_06268_amd import workloads as W
from parity_util import assert_same_state, make_pair

pytestmark = pytest.mark.gpu

SIZES = [(2, 3), (4, 4), (6, 5), (10, 3), (12, 2), (14, 4), (18, 3), (20, 2), (22, 2), (24, 3), (26, 2), (28, 3), (36, 2),
         (40, 3), (48, 2), (52, 2), (12, 40), (24, 30), (18, 33), (36, 25), (40, 25), (60, 1), (72, 1)]


@pytest.mark.parametrize("L,R", SIZES)
def test_chain_matches_oracle(rfim_mod, oracle_mod, L, R):
    f = W.bimodal_fields(L, [95, L])
    T = W.linear_temps(R, 2.0, 2.0 + 0.002 * (R - 1) * (64 / L) ** 1.5) if R > 1 else np.array([2.0])
    g, o = make_pair(rfim_mod, oracle_mod, L, R, 1.0, 1.5, f, T, seed=L, R_cap=R + 2)
    for n, every in ((11, 4), (5, 7), (3, 0), (2, 1)):
        g.sweep(n, every)
        o.sweep(n, every)
    assert_same_state(g, o, "L=%d" % L)
    g.adapt_temps(1, 8, 4, 1.1, 2, R + 2)
    o.adapt_temps(1, 8, 4, 1.1, 2, R + 2)
    g.sweep(9, 4)
    o.sweep(9, 4)
    assert_same_state(g, o, "L=%d after insertion" % L)
    g.close()
    o.close()


@pytest.mark.parametrize("L,R", [(6, 5), (12, 4), (22, 3), (24, 3), (26, 2), (28, 3), (40, 3), (48, 2)])
def test_continuous_decisions_match_oracle(rfim_mod, oracle_mod, L, R):
    f = W.gaussian_fields(L, [96, L])
    T = W.geometric_temps(R, 1.0, 6.0)
    g, o = make_pair(rfim_mod, oracle_mod, L, R, 1.0, 2.0, f, T, seed=L)
    for rep in range(2):
        s = W.random_spins(R, L, [97, L, rep])
        g.set_spins(s)
        o.set_spins(s)
        g.sweep(1, 0)
        o.sweep(1, 0)
        assert int((g.spins() != o.spins()).sum()) <= 1
    g.sweep(12, 5)
    E, obs, perm = g.energies(), g.observables(), g.perm()
    assert np.array_equal(np.sort(perm), np.arange(R)) and np.all(obs[:, 0] == 2)
    s = g.spins()
    g.set_spins(s)
    assert np.allclose(g.energies(), E, rtol=1e-12, atol=1e-9)
    g.close()
    o.close()


@pytest.mark.parametrize("L,R", [(12, 40), (12, 2), (20, 3), (28, 60), (28, 3), (36, 25), (36, 2), (40, 25), (40, 3), (48, 5),
                                 (52, 2), (60, 3), (72, 2), (22, 3), (26, 2), (90, 1)])
def test_sampled_energies_are_those_of_the_configurations(rfim_mod, L, R):
    """The energy that the exchange step samples after a sweep (from the sweep
    kernels' own sums where they have them) against the energies read of the
    same configurations, and those against sums in another order: FP64 sums of
    4 N terms of size 1, J and h |f|, so within 4 N eps of their absolute sum
    (exact for +-1 fields)."""
    N = L ** 3
    for kind, f in (("b", W.bimodal_fields(L, [99, L])), ("g", W.gaussian_fields(L, [99, L]))):
        g = rfim_mod.Rfim(L, R, 1.0, 1.5, f, W.linear_temps(R, 2.0, 5.0) if R > 1 else np.array([2.0]), seed=L)
        for n, every in ((3, 3), (5, 8), (1, 1)):
            g.reset_observables()
            g.sweep(n, every)
            obs, E = g.observables(), g.energies()
            bound = 4 * N * 2.0 ** -53 * (3 * N + 1.5 * float(np.abs(f).sum(dtype=np.float64))) if kind == "g" else 0.0
            assert np.all(obs[:, 0] == 1) and np.abs(obs[:, 1] - E).max() <= bound
            assert np.array_equal(obs[:, 3], np.abs(g.magnetizations()))
            s, perm = g.spins(), g.perm()
            assert abs(E[R - 1] - energy_numpy(s[perm[R - 1]], f, L, 1.0, 1.5)[0]) <= bound
        g.close()


def philox_numpy(c0, c1, c2, c3, key):
    """Philox4x32-10 of many counters, uint64 arrays of 32-bit words."""
    M = np.uint64(0xFFFFFFFF)
    c = [np.broadcast_to(np.asarray(v, dtype=np.uint64), np.shape(c0)) for v in (c0, c1, c2, c3)]
    k0, k1 = key & 0xFFFFFFFF, key >> 32
    for _ in range(10):
        a, b = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & M, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & M]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return np.stack(c, axis=-1)


def test_more_sites_than_one_launch_takes(rfim_mod):
    """R L^3 > 2^35 (35 GB of spins): a half-sweep is two launches, from
    replica 38836 on (of 432 workgroups of 256 threads each).  So cold that a
    spin flips only where its energy does not rise, each replica ends where its
    random start leads."""
    L, R, seed = 96, 40000, 5
    f = W.bimodal_fields(L, [98, L])
    g = rfim_mod.Rfim(L, R, 1.0, 1.5, f, np.linspace(0.010, 0.011, R), seed=seed)
    g.sweep(1, 0)
    E, M = g.energies(), g.magnetizations()
    g.close()
    for r in (0, 38835, 38836, R - 1):
        w = philox_numpy(np.arange(L ** 3 // 4), 0, r, 1 << 28, seed)
        s = quench_numpy(np.where(w.reshape(-1) >= 1 << 31, 1, -1).astype(np.int8), f, L, 1.0, 1.5, 1)
        assert E[r] == energy_numpy(s, f, L, 1.0, 1.5)[0] and M[r] == int(s.sum(dtype=np.int64)), r
