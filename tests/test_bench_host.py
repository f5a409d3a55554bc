"""bench.py's per-kernel figures (no GPU needed): rates and fractions are those
of the work a launch does, however many lattices it covers."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("valid", [False, True])
def test_figures_do_not_depend_on_the_slices(bench, valid):
    N, lattices, sweeps = 16 * 128 ** 3, 5, 10
    us = {"local": 110.0, "unite": 85.0, "flip": 70.0}  # per lattice

    def bounds(launches):  # per sweep, covering the five lattices together
        kt = {k: (launches * sweeps, v * lattices * sweeps * 1e-3) for k, v in us.items()}
        kt["persist"] = (0, 0.0)
        return bench.kernel_bounds(kt, N, lattices * sweeps, 9.0e5, 8.5e5, 2.3e10, 5.0e3, valid)

    one, two, five = bounds(1), bounds(2), bounds(5)
    for k in us:
        assert two[k]["lattices_per_launch"] == 2.5 and five[k]["lattices_per_launch"] == 1.0
        for f in five[k]:
            if "frac" in f or "per_s" in f or f in ("bound", "achieved_GBps", "valu_per_wave", "salu_per_wave"):
                assert two[k][f] == pytest.approx(five[k][f]) and one[k][f] == pytest.approx(five[k][f]), (k, f)
        assert two[k]["us"] == pytest.approx(2.5 * us[k])
    assert five["local"]["hbm_alg_frac"] == pytest.approx(5.0 * N / 110e-6 / 8e12)
    assert two["unite"]["achieved_cas_per_s"] == pytest.approx(9.0e5 / 85e-6)
    assert two["unite"]["cas_per_launch"] == 2250000
    assert five["flip"]["hbm_alg_frac"] == pytest.approx(6.0 * N / 70e-6 / 8e12)


def test_launch_traffic(bench):
    t = bench.MEASURED_TRAFFIC["local"]
    assert bench.launch_traffic("local", 2.5, True) == pytest.approx(2.5 * t)
    assert bench.launch_traffic("local", 1.0, False) is None and bench.launch_traffic("persist", 1.0, True) is None
