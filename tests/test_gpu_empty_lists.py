"""Tiles whose crossing lists are empty (infinite temperature: no active bond)
or hold a pair here and there: the unite pass leaves an empty list at once, in
per-sweep and persistent launches, beside replicas whose lists are long.
Ising records, spins and labels bit for bit as the oracle's, O(n) spins and
labels bit for bit and records within 1e-5."""
import sys

import numpy as np
import pytest

import oracle
from paper_1612_08312_amd import pyrosw

pytestmark = pytest.mark.gpu

INF = float("inf")


@pytest.mark.parametrize("model,temps", [(1, (INF, 400.0, 4.2)), (2, (400.0, INF, 2.0)), (3, (2.0, 400.0, INF))])
@pytest.mark.parametrize("shape", [pyrosw.PYRO_TILE_8x4x4, pyrosw.PYRO_TILE_8x8x8])
@pytest.mark.parametrize("persistent", [False, True])
def test_empty_and_short_lists(model, temps, shape, persistent):
    if persistent and model != 1:
        return
    print("GPU case: empty crossing lists", model, shape, persistent, file=sys.stderr, flush=True)
    cfgs = [dict(L=L, model=model, T=T, seed=61 + k, start=1) for k, (L, T) in enumerate(zip((17, 16, 20), temps))]
    lats = [pyrosw.Lattice(**c) for c in cfgs]
    group = pyrosw.Group(lats)
    group.set_tile_shape(model, shape)
    if persistent:
        group.set_mode(pyrosw.PYRO_MODE_PERSISTENT)
    group.sweep(3)
    group.sweep(2)
    for c, lt in zip(cfgs, lats):
        o = oracle.Oracle(**c)
        rec, ref = lt.moments(), o.sweep(5)
        np.testing.assert_array_equal(lt.spins(), o.spins())
        np.testing.assert_array_equal(lt.labels(), o.labels())
        for f in ("sweep", "bond_sum", "M_int", "E", "M", "m2", "m4"):
            if model == 1:
                np.testing.assert_array_equal(rec[f], ref[f], err_msg=f)
            else:
                np.testing.assert_allclose(rec[f], ref[f], rtol=1e-5, atol=1e-5 * np.abs(ref[f]).max(), err_msg=f)
    group.close()
    for lt in lats:
        lt.close()
