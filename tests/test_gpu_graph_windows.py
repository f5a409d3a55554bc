"""The bond-table path on both sides of the sizes where its windows change,
and a table whose window draws its Philox blocks in several chunks: records,
spins and labels against the oracle (Ising bit for bit; XY spins and labels
bit for bit, records within 1e-5, FP64 sums in another order)."""
import sys

import numpy as np
import pytest

import oracle
from paper_1612_08312_amd import pyrosw

pytestmark = pytest.mark.gpu


def check(g, o, sweeps, model):
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


@pytest.mark.parametrize("L,model,T", [(50, 1, 4.511524), (51, 1, 4.511524), (51, 2, 2.20182), (81, 1, 4.511524)])
def test_simple_cubic_of_each_window_size(L, model, T):
    print("GPU case: simple cubic window sizes", L, model, file=sys.stderr, flush=True)
    g = pyrosw.Graph(pyrosw.simple_cubic_bonds(L), L ** 3, model, T, seed=9)
    check(g, oracle.Oracle(L=L, model=model, T=T, seed=9, start=1, lattice="sc"), 3, model)


@pytest.mark.parametrize("per_window", [700, 16384, 16385, 40000])
def test_windows_of_many_draws(per_window):
    """Two dense clumps of 512 sites: 44 to 2500 blocks of 16 draws per window
    (1024 are kept at a time), and single bonds left over."""
    print("GPU case: draws per window", per_window, file=sys.stderr, flush=True)
    rng = np.random.default_rng(per_window)
    a, b = [], []
    for lo in (0, 512):
        i = rng.integers(0, 512, per_window)
        a.append(lo + i)
        b.append(lo + (i + rng.integers(1, 512, per_window)) % 512)
    a.append(np.arange(300))
    b.append(np.arange(300) + 700)
    a, b = np.concatenate(a).astype(np.int32), np.concatenate(b).astype(np.int32)
    T = per_window / 100.0
    g = pyrosw.Graph((a, b), 1030, 1, T, seed=4)
    check(g, oracle.Oracle(model=1, T=T, seed=4, start=1, lattice="edges", edges=(a, b), n_sites=1030), 12, 1)
