"""Groups of several models: the passes that their chains share in one launch
give every member the sweeps it has alone (the arithmetic of a tile does not
depend on its launch)."""
import numpy as np
import pytest

from paper_1612_08312_amd import pyrosw

pytestmark = pytest.mark.gpu

T = {1: 4.21394, 2: 2.0285, 3: 1.31695}


# (model, L): the two O(n) chains alone with one tile shape and with two
# (L >= 48 takes 8x8x4 tiles), each with an Ising chain, and all three.
@pytest.mark.parametrize("members", [
    ((2, 9), (3, 16)), ((3, 5), (2, 16), (3, 24)), ((2, 48), (3, 8)),
    ((1, 10), (2, 17)), ((1, 8), (3, 12)), ((1, 16), (2, 8), (3, 8)), ((1, 1), (2, 1), (3, 1)), ((1, 49), (2, 16), (3, 50)),
])
@pytest.mark.parametrize("slices", [1, 2])
def test_shared_passes_equal_lone_sweeps(members, slices):
    def make():
        return [pyrosw.Lattice(L=L, model=m, T=T[m], seed=11 + k) for k, (m, L) in enumerate(members)]

    counts = [6 - k for k in range(len(members))]
    together = make()
    group = pyrosw.Group(together)
    group.set_slices(min(slices, len(members)))
    group.sweep(0, counts)
    for lt, alone, n in zip(together, make(), counts):
        alone.sweep(n)
        a, b = lt.moments(), alone.moments()
        for f in ("sweep", "bond_sum", "M_int", "M", "m2", "m4"):
            np.testing.assert_array_equal(a[f], b[f])
        # an earlier autotuning of such a group may have chosen another tile
        # shape, which orders the FP64 sum of an O(n) energy differently
        np.testing.assert_allclose(a["E"], b["E"], rtol=1e-13, atol=0)
        np.testing.assert_array_equal(lt.spins(), alone.spins())
