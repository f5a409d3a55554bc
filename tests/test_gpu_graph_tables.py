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


def window_of(n):
    """Sites per window of a large table, the library's rule restated."""
    return 4096 if n >= 2 ** 20 else 2048 if n >= 2 ** 19 else 1024 if n >= 2 ** 17 else 512


def permuted(table, seed=3):
    """The same bonds in random order: the 16 bonds of a Philox block lie in
    windows of their own, so every bond draws its own."""
    p = np.random.default_rng(seed).permutation(len(table[0]))
    return np.ascontiguousarray(table[0][p]), np.ascontiguousarray(table[1][p])


# Both sides of the sizes where the windows change (2^19 = 524,288 lies between
# L = 80 and 81, 2^20 = 1,048,576 between 101 and 102), with shared and with
# own draws, and the O(n) pass that projects in the window.
@pytest.mark.parametrize("L,model,T,order", [
    (80, 1, 4.511524, "rows"), (101, 1, 4.511524, "rows"), (102, 1, 4.511524, "rows"), (81, 1, 4.511524, "permuted"),
    (102, 1, 4.511524, "permuted"), (80, 2, 2.20182, "rows"), (81, 2, 2.20182, "rows"), (102, 2, 2.20182, "rows"),
    (81, 3, 1.443, "rows")])
def test_simple_cubic_of_every_window_size(L, model, T, order):
    table = tuple(np.asarray(x, np.int32) for x in pyrosw.simple_cubic_bonds(L))
    check(table if order == "rows" else permuted(table), L ** 3, model, T, 3)


def cut(n, a, b, window, ball):
    """Bonds between windows: balls grown breadth first from the smallest free
    site, or runs of consecutive indices."""
    if not ball:
        return int(np.sum(a // window != b // window))
    # neighbours in the order of the bonds: bond k lists its second end at its
    # first end and its first end at its second
    src = np.concatenate([a, b])
    dst = np.concatenate([b, a])
    k = np.concatenate([np.arange(len(a))] * 2)
    order = np.lexsort((k, src))
    dst = dst[order].tolist()
    off = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).tolist()
    win = [-1] * n
    w = fill = nxt = taken = 0
    while taken < n:
        while win[nxt] >= 0:
            nxt += 1
        queue = [nxt]
        win[nxt] = w
        taken, fill = taken + 1, fill + 1
        h = 0
        while h < len(queue) and fill < window:
            x = queue[h]
            h += 1
            for y in dst[off[x]:off[x + 1]]:
                if win[y] < 0:
                    win[y] = w
                    queue.append(y)
                    taken, fill = taken + 1, fill + 1
                    if fill == window:
                        break
        if fill == window:
            w, fill = w + 1, 0
    win = np.asarray(win)
    return int(np.sum(win[a] != win[b]))


@pytest.mark.parametrize("lattice,model,L,T,ball", [("sc", 1, 48, 4.511524, True), ("sc", 2, 40, 2.20182, True),
                                                    ("sc", 1, 52, 4.511524, True), ("pyro", 1, 12, 4.2139, True),
                                                    ("ring", 1, 60000, 0.5, False)])
def test_windows_of_either_kind(lattice, model, L, T, ball):
    """Tables whose windows are breadth-first balls, and consecutive runs, at
    the window size that the library uses for them."""
    if lattice == "ring":
        table, n = ring(L), L
    else:
        table = pyrosw.simple_cubic_bonds(L) if lattice == "sc" else pyrosw.pyro_sw_bonds(L)
        n = L ** 3 if lattice == "sc" else 16 * L ** 3
    a, b = (np.asarray(x, np.int64) for x in table)
    w = window_of(n)
    assert (cut(n, a, b, w, True) < cut(n, a, b, w, False)) == ball
    check(tuple(np.asarray(x, np.int32) for x in table), n, model, T, 12)
