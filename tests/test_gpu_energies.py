"""Energies, bond sums, field sums and magnetisations of a state at rest
(rfim_components, rfim_energies) against the roll formulation, for every form
of the energy kernel: rows of 4-dword and 1-dword chunks, rows that end
inside a dword, and bit storage."""
import numpy as np
import pytest

from helpers import energy_numpy
from paper_1508_06268_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,R", [(2, 3), (6, 5), (8, 16), (12, 1), (16, 5), (24, 4), (32, 7), (40, 2), (50, 2), (64, 5),
                                 (96, 2), (128, 2)])
@pytest.mark.parametrize("kind", ["b", "g"])
def test_components_match_numpy(rfim_mod, L, R, kind):
    f = W.bimodal_fields(L, [81, L]) if kind == "b" else W.gaussian_fields(L, [81, L])
    g = rfim_mod.Rfim(L, R, 1.0, 1.5, f, W.linear_temps(R, 1.5, 4.0), seed=3)
    g.sweep(4, 2)
    for storage in ([rfim_mod.rfim.SPINS_BITS, rfim_mod.rfim.SPINS_BYTES] if L in (64, 128) else [None]):
        if storage is not None:
            g.set_spin_storage(storage)
        s, perm = g.spins(), list(g.perm())
        B, F, M = g.components()
        E, Ms = g.energies(), g.magnetizations()
        for r in range(R):
            want, bonds = energy_numpy(s[r], f, L, 1.0, 1.5)
            slot = perm.index(r)
            assert B[r] == bonds and M[r] == s[r].sum() == Ms[slot]
            if kind == "b":
                assert E[slot] == want
            else:       # FP64 sums of N terms in another order
                assert np.isclose(E[slot], want, rtol=1e-12, atol=1e-9)
                assert np.isclose(F[r], float((f.astype(np.float64) * s[r]).sum()), rtol=1e-11, atol=1e-9)
    g.close()
