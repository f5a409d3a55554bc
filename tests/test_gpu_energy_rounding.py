"""Rounding of the O(n) energy in the tile pass: on one cell (L = 1) ordered
enough for the running sum to grow, the FP64 sum over its 48 bonds is no
further from the exact sum than one rounding per bond at the size of the
running sum, on the mean over 300 states."""
import math
import sys

import numpy as np
import pytest

from paper_1612_08312_amd import pyrosw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,T", [(2, 0.1), (2, 1.0), (3, 0.1), (3, 1.0)])
def test_cell_energy_rounds_no_more_than_once_per_bond(model, T):
    print("GPU case: energy rounding, model", model, "T", T, file=sys.stderr, flush=True)
    n = 300
    kw = dict(L=1, model=model, T=T, seed=71, start=0)
    lt, states = pyrosw.Lattice(**kw), pyrosw.Lattice(**kw)
    lt.sweep(n + 1)  # every record but the last takes its energy from the next sweep's tile pass
    E = lt.moments()["E"][:n]
    a, b = (np.asarray(x, np.int64) for x in pyrosw.pyro_sw_bonds(1))
    got, once = [], []
    for k in range(n):
        states.sweep(1)
        s = states.spins().reshape(model, -1).astype(np.float64)
        p = s[:, a] * s[:, b]  # products of FP32 numbers are exact in FP64
        exact = math.fsum(p.ravel())
        total = 0.0
        for bond in p.T:
            dot = 0.0
            for v in bond:
                dot += v
            total += dot
        got.append(-E[k] - exact)
        once.append(total - exact)
    rms = [float(np.sqrt(np.mean(np.square(v)))) for v in (got, once)]
    print("rms error %.2e, one rounding per bond %.2e" % tuple(rms), file=sys.stderr, flush=True)
    assert np.max(np.abs(got)) < 1e-12 and rms[0] <= rms[1]
    lt.close()
    states.close()
