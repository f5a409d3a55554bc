"""Bond tables on each side of the rules that choose how they are swept:
spins and labels equal the oracle's bit for bit, records too for Ising (O(n)
records within 1e-5, FP64 sums in another order)."""
import sys

import numpy as np
import pytest

import oracle
from paper_1612_08312_amd import pyrosw

pytestmark = pytest.mark.gpu


def random_table(n, bonds, seed=5):
    rng = np.random.default_rng(seed)
    a = rng.integers(0, n, bonds)
    return a.astype(np.int32), ((a + rng.integers(1, n, bonds)) % n).astype(np.int32)


def check(table, n, model, T, sweeps):
    print("GPU case: bond table, %d sites, %d bonds, model %d" % (n, len(table[0]), model), file=sys.stderr, flush=True)
    g = pyrosw.Graph(table, n, model, T, seed=17)
    o = oracle.Oracle(model=model, T=T, seed=17, start=1, lattice="edges", edges=table, n_sites=n)
    g.sweep(sweeps)
    rec, ref = g.moments(), o.sweep(sweeps)
    np.testing.assert_array_equal(g.labels(), o.labels())
    np.testing.assert_array_equal(g.spins(), o.spins())
    for f in ("sweep", "bond_sum", "M_int", "E", "M", "m2", "m4"):
        if model == 1:
            np.testing.assert_array_equal(rec[f], ref[f], err_msg=f)
        else:
            np.testing.assert_allclose(rec[f], ref[f], rtol=1e-5, atol=1e-5 * np.abs(ref[f]).max(), err_msg=f)
    g.close()


@pytest.mark.parametrize("n,model,T", [(2 ** 19 - 1, 2, 0.8), (2 ** 19, 2, 0.8), (2 ** 19 + 1, 3, 0.5)])
def test_projections_in_site_order(n, model, T):
    """Random tables from 2^19 sites on write the projections in a pass of
    their own."""
    check(random_table(n, 2 * n), n, model, T, 4)


def ring(n):
    i = np.arange(n, dtype=np.int32)
    return i, ((i + 1) % n).astype(np.int32)


# One window for a small graph of few bonds, most of them cut, else windows of
# 512 sites: at most 8192 bonds up to 1024 sites, 7168 up to 2048, 5120 up to
# 4096.  (sites, bonds; None: a ring, which windows of 512 hardly cut)
@pytest.mark.parametrize("model", [1, 2])
@pytest.mark.parametrize("n,bonds", [(513, 900), (1024, 8192), (1024, 8193), (1025, 7168), (2048, 7169), (2049, 5120),
                                     (4096, 5120), (4096, 5121), (4097, 3000), (600, None), (3000, None)])
def test_small_tables_of_one_window_or_several(n, bonds, model):
    table = ring(n) if bonds is None else random_table(n, bonds, n)
    check(table, n, model, 2.0 * len(table[0]) / n / (1 if model == 1 else 3), 25)
