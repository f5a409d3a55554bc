"""Records across a change of the way a lattice is swept, read once at the end:
LDS-resident sweeps in a group followed by tiled ones (alone, in per-sweep
graphs, persistent), which must leave the resident sweeps' last record as it
is, and the same after tiled sweeps whose last record is still pending.
Every record, spin and label equals the oracle's bit for bit."""
import sys

import numpy as np
import pytest

import oracle
from paper_1612_08312_amd import pyrosw

pytestmark = pytest.mark.gpu

GRAPH, PERSIST = pyrosw.PYRO_MODE_GRAPH, pyrosw.PYRO_MODE_PERSISTENT
T = 4.2139


def sweep_alone(lats, group, n):
    for lt in lats:
        if lt.L <= 13:  # a lattice this small would sweep LDS-resident
            lt.set_tile_shape(pyrosw.PYRO_TILE_8x4x4)
        lt.sweep(n)


def sweep_graph(lats, group, n):
    group.set_mode(GRAPH, False)
    group.sweep(n)


def sweep_persistent(lats, group, n):
    group.set_mode(PERSIST, False)
    group.sweep(n)


def sweep_resident(lats, group, n):
    group.set_mode(GRAPH, True)
    group.sweep(n)


WAYS = {"alone": sweep_alone, "graph": sweep_graph, "persistent": sweep_persistent, "resident": sweep_resident}


@pytest.mark.parametrize("L", [8, 14, 16])
@pytest.mark.parametrize("ways", [("resident", "alone"), ("resident", "graph"), ("resident", "persistent"),
                                  ("graph", "resident", "graph"), ("persistent", "resident", "persistent"),
                                  ("graph", "persistent", "alone", "resident", "alone")])
def test_records_across_modes(L, ways):
    print("GPU case: records across modes", L, ways, file=sys.stderr, flush=True)
    cfgs = [dict(L=L, model=1, T=T, seed=41, start=1), dict(L=L, model=1, T=3.9, seed=42, start=1)]
    lats = [pyrosw.Lattice(**c) for c in cfgs]
    group = pyrosw.Group(lats)
    for k, way in enumerate(ways):
        WAYS[way](lats, group, 3 + k)
    total = sum(3 + k for k in range(len(ways)))
    for c, lt in zip(cfgs, lats):
        o = oracle.Oracle(**c)
        rec, ref = lt.moments(), o.sweep(total)
        for f in ("sweep", "bond_sum", "M_int", "E", "M", "m2", "m4"):
            np.testing.assert_array_equal(rec[f], ref[f], err_msg=f)
        np.testing.assert_array_equal(lt.spins(), o.spins())
        np.testing.assert_array_equal(lt.labels(), o.labels())
    group.close()
    for lt in lats:
        lt.close()


def test_a_member_that_sits_out_a_resident_call():
    """A member with no sweep in a call keeps its pending record."""
    print("GPU case: member without sweeps", file=sys.stderr, flush=True)
    cfgs = [dict(L=10, model=1, T=T, seed=43 + k, start=1) for k in range(2)]
    lats = [pyrosw.Lattice(**c) for c in cfgs]
    group = pyrosw.Group(lats)
    counts = [0, 0]
    for way, n in ((GRAPH, [2, 3]), (True, [0, 4]), (PERSIST, [0, 2]), (GRAPH, [3, 0]), (True, [2, 2]), (GRAPH, [0, 1])):
        group.set_mode(GRAPH if way is True else way, way is True)
        group.sweep(0, n)
        counts = [a + b for a, b in zip(counts, n)]
    for c, lt, n in zip(cfgs, lats, counts):
        rec, ref = lt.moments(), oracle.Oracle(**c).sweep(n)
        for f in ("sweep", "bond_sum", "M_int", "E", "M", "m2", "m4"):
            np.testing.assert_array_equal(rec[f], ref[f], err_msg=f)
    group.close()
    for lt in lats:
        lt.close()
