"""Lattice sizes that are not powers of two (and L = 2, 4): the LDS-resident
form, boxes (slabs and whole replicas), the streaming half-sweeps, rows of
whole dwords and rows that end inside one.  +-1 fields follow the oracle bit for bit; of one sweep's decisions with
continuous fields at most one differs (they are FP32 on the device: about 1 in
3e7)."""
import numpy as np
import pytest

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
