"""Lone small Ising lattices, which sweep LDS-resident (L <= 13): every record,
spin and label equals the oracle's bit for bit, on both sides of the sizes
where a thread takes one tetrahedron more, at the temperatures where no byte
ties or every bond is active, after tiled sweeps whose last record is still
pending, and against the tiled sweep of the same lattice."""
import sys

import numpy as np
import pytest

import oracle
from paper_1612_08312_amd import pyrosw

pytestmark = pytest.mark.gpu


def same(g, rec, o, orec):
    for f in ("sweep", "bond_sum", "M_int", "E", "M", "m2", "m4"):
        np.testing.assert_array_equal(rec[f], orec[f], err_msg=f)
    np.testing.assert_array_equal(g.spins(), o.spins())
    np.testing.assert_array_equal(g.labels(), o.labels())


@pytest.mark.parametrize("L,T", [(1, 4.2139), (2, 4.2139), (4, 0.05), (4, float("inf")), (6, 4.2139), (7, 4.2139), (8, 4.2139),
                                 (9, 4.2139), (10, 1.0), (12, 4.2139), (13, 4.2139), (14, 4.2139)])
def test_small_lattices_equal_the_oracle(L, T):
    print("GPU case: small lattice", L, T, file=sys.stderr, flush=True)
    sweeps = (1, 12, 2)  # L = 13 crosses between the tiled and the resident sweep
    for tiled in (False, True):
        g = pyrosw.Lattice(L=L, model=1, T=T, seed=5, start=1)
        o = oracle.Oracle(L=L, model=1, T=T, seed=5, start=1)
        if tiled:
            g.set_tile_shape(pyrosw.PYRO_TILE_8x4x4)
        for n in sweeps:
            g.sweep(n)
        same(g, g.moments(), o, o.sweep(sum(sweeps)))
        g.close()


@pytest.mark.parametrize("L", [3, 8, 12])
def test_resident_sweeps_after_tiled_ones(L):
    """Timed sweeps are tiled and leave their last record's sums pending."""
    print("GPU case: tiled, resident, tiled", L, file=sys.stderr, flush=True)
    g = pyrosw.Lattice(L=L, model=1, T=4.2139, seed=6, start=1)
    o = oracle.Oracle(L=L, model=1, T=4.2139, seed=6, start=1)
    for mask, n in ((-1, 3), (0, 4), (-1, 2), (0, 1)):
        pyrosw.pyro_sw_set_timing(g.h, mask)
        g.sweep(n)
    same(g, g.moments(), o, o.sweep(10))
    g.close()


@pytest.mark.parametrize("first,second", [(2, 3), (3, 1)])
def test_pending_record_across_tile_shapes(first, second):
    """A record whose magnetisation was left by one tile shape and is summed
    after sweeps, or at a drain, under another."""
    print("GPU case: tile shapes", first, second, file=sys.stderr, flush=True)
    g = pyrosw.Lattice(L=17, model=1, T=4.2139, seed=7, start=1)
    o = oracle.Oracle(L=17, model=1, T=4.2139, seed=7, start=1)
    g.set_tile_shape(first)
    g.sweep(2)
    g.set_tile_shape(second)
    g.sweep(2)
    g.set_tile_shape(first)
    same(g, g.moments(), o, o.sweep(4))
    g.close()
