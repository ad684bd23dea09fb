"""Which iteration kernel a step is launched with: the tests that compare the
split kernel with the other have the split kernel on one side and only there."""
import numpy as np
import pytest

from paper_2308_01654_amd import scenes
from tests import test_gpu_parity as parity

pytestmark = pytest.mark.gpu

SPLIT = 2


def _mppi():
    from paper_2308_01654_amd import mppi
    mppi.load()
    return mppi


def _shapes(test):
    """(lanes, K, T, circles, waypoints, overrides) of a parity test's cases."""
    for mark in test.pytestmark:
        if mark.name == "parametrize" and "K" in mark.args[0]:
            names = mark.args[0].split(",")
            for v in mark.args[1]:
                c = dict(zip(names, v))
                yield (c.get("lanes", 16), c["K"], c["T"], c["n_c"], c.get("n_wp", 333), c["over"])


def _kernels(K, T, n_c, n_wp, over, lanes, cull=True):
    mppi = _mppi()
    rng = np.random.Generator(np.random.PCG64(K + T))
    sc = scenes.tiny(K=K, T=T, n_c=0, seed=3)
    p = dict(scenes.params(K=K, T=T, dt=0.05, v_max=15.0, seed=7), **over)
    out = []
    for occ in (-1, 0):
        with mppi.Planner(p, lanes=lanes) as pl:
            with pytest.raises(mppi.MppiError) as e:
                pl.kernel()
            assert e.value.status == mppi.E_NOT_READY
            pl.set_occupancy(occ)
            pl.set_culling(cull)
            pl.step(sc["x0"], parity._bent(n_wp), scenes.sine_circles(rng, n_c, 0.0, 60.0))
            out.append(pl.kernel())
    return out


@pytest.mark.parametrize("test", [parity.test_split_kernel_bit_identical,
                                  parity.test_split_kernel_at_8_and_4_lanes_bit_identical])
def test_parity_cases_run_the_split_kernel(test):
    n = 0
    for lanes, K, T, n_c, n_wp, over in _shapes(test):
        assert _kernels(K, T, n_c, n_wp, over, lanes) == [SPLIT, 0], (lanes, K, T, n_c)
        n += 1
    assert n >= 17


@pytest.mark.parametrize("n_c", [65, 1024])
def test_grouped_circles_run_the_split_kernel(n_c):
    """Scenes of test_grouped_circles_bit_identical, with culling and without."""
    assert _kernels(200, 60, n_c, 221, {}, 16) == [SPLIT, 0]
    assert _kernels(200, 60, n_c, 221, {}, 16, cull=False) == [0, 0]
