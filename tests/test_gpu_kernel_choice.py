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


# On either side of each line of the rule: 512 tiles (two per compute unit) and
# more, alone and in a batch of n; horizons; circles that are all listed (up to
# 64), more, none; per-step weights.  At 4 lanes and 90 steps the tiles do not keep
# their perturbations.
@pytest.mark.parametrize("lanes,n,K,T,n_c,ps,split", [
    (16, 1, 8208, 16, 12, 0, 1), (16, 2, 4096, 16, 12, 0, 1), (16, 3, 2736, 47, 12, 0, 0),
    (16, 3, 2736, 48, 12, 0, 1), (16, 3, 2736, 16, 0, 0, 1), (16, 3, 2736, 63, 65, 1, 0),
    (16, 3, 2736, 64, 65, 1, 1), (16, 2, 4096, 16, 12, 1, 1),
    (8, 1, 16384, 24, 12, 0, 1), (8, 1, 16384, 24, 12, 1, 0), (8, 1, 16416, 31, 12, 0, 0),
    (8, 1, 16416, 32, 64, 0, 1), (8, 1, 16416, 79, 0, 0, 0), (8, 1, 16416, 80, 0, 0, 1),
    (8, 1, 16416, 79, 65, 0, 0),
    (8, 1, 16416, 80, 65, 0, 1), (8, 2, 8192, 24, 12, 0, 1), (8, 2, 8224, 99, 12, 0, 0),
    (8, 2, 8224, 100, 12, 0, 1), (8, 2, 8224, 100, 0, 0, 0), (8, 2, 8224, 127, 65, 0, 0),
    (8, 2, 8224, 128, 65, 0, 1),
    (4, 1, 32768, 63, 12, 0, 0), (4, 1, 32768, 64, 12, 0, 1), (4, 1, 32768, 64, 0, 0, 0),
    (4, 1, 32832, 64, 12, 0, 1), (4, 1, 32832, 64, 65, 0, 0), (4, 1, 32832, 90, 12, 0, 0),
    (4, 1, 32832, 128, 65, 0, 1), (4, 2, 16448, 149, 12, 0, 0), (4, 2, 16448, 150, 12, 0, 1),
    (2, 1, 2048, 100, 12, 0, 0),
])
def test_rule_of_the_split_kernel(lanes, n, K, T, n_c, ps, split):
    """The kernel that is launched, with the bits of the other one."""
    _check(lanes, n, K, T, n_c, ps, split, scenes.tiny()["waypoints"])


# Paths around 64 chunks of 8 waypoints and the lines past them, in launches of few
# tiles and of more, with circles that are listed and in groups
@pytest.mark.parametrize("lanes,K,T,n_c,n_wp,split", [
    (16, 300, 20, 12, 1536, 1), (16, 300, 20, 12, 1537, 0), (16, 300, 20, 65, 2048, 1),
    (8, 300, 20, 12, 640, 1), (8, 300, 20, 0, 641, 0), (8, 300, 20, 65, 2048, 1),
    (8, 300, 100, 12, 1024, 1), (8, 300, 100, 12, 1025, 0),
    (16, 8208, 20, 12, 512, 1), (16, 8208, 20, 12, 513, 0), (16, 8208, 20, 65, 1024, 1),
    (16, 8208, 20, 65, 1025, 0), (16, 8208, 100, 65, 1536, 1), (16, 8208, 100, 65, 1537, 0),
    (16, 8208, 150, 65, 2048, 1), (16, 8208, 200, 12, 640, 1), (16, 8208, 200, 12, 641, 0),
    (16, 8208, 199, 12, 640, 0), (8, 16416, 200, 0, 513, 0),
])
def test_rule_of_the_split_kernel_for_long_paths(lanes, K, T, n_c, n_wp, split):
    _check(lanes, 1, K, T, n_c, 0, split, parity._bent(n_wp, 0.5))


def _check(lanes, n, K, T, n_c, ps, split, waypoints):
    mppi = _mppi()
    rng = np.random.Generator(np.random.PCG64(T))
    sc = dict(scenes.tiny(K=K, T=T, n_c=0, seed=3), waypoints=waypoints)
    p = dict(sc["params"], per_step=ps)
    ci = scenes.sine_circles(rng, n_c, 0.0, 60.0)
    print("  case:", lanes, n, K, T, n_c, ps, len(waypoints), flush=True)
    lead = mppi.Planner(p, lanes=lanes)
    pls = [lead] + [mppi.Planner(p, lanes=lanes, hip_stream=lead.stream()) for _ in range(n - 1)]
    try:
        if n == 1:
            lead.step(sc["x0"], sc["waypoints"], ci)
        else:
            mppi.step_batch(pls, np.array([sc["x0"]] * n), [(sc["waypoints"], ci)] * n)
        assert [pl.kernel() == SPLIT for pl in pls] == [bool(split)] * n
        with mppi.Planner(p, lanes=lanes) as ref:
            ref.set_occupancy(0)
            ref.step(sc["x0"], sc["waypoints"], ci)
            assert ref.kernel() == 0
            assert np.array_equal(pls[-1].costs(), ref.costs())
            assert np.array_equal(pls[-1].controls(), ref.controls())
    finally:
        for pl in reversed(pls):
            pl.close()


@pytest.mark.parametrize("shapes,asked,kernels", [
    # few tiles for either kernel go with the many of the other
    ([(4096, 40), (8192, 100), (8192, 100), (2048, 60)], {}, [SPLIT] * 4),
    ([(8192, 20), (8192, 24), (1024, 100), (2048, 20)], {}, [0] * 4),
    # each its own where both are many; a compilation asked for is kept
    ([(16400, 20), (16400, 100)], {}, [0, SPLIT]),
    ([(4096, 40), (8192, 100), (8192, 100)], {0: 0, 1: 1}, [0, 1, SPLIT]),
])
def test_few_tiles_of_a_batch_go_with_the_others(shapes, asked, kernels):
    """Kernels of a batch of uneven instances at 16 lanes per sample; each has its
    bits from alone."""
    mppi = _mppi()
    insts = [scenes.tiny(K=K, T=T, n_c=9, seed=i) for i, (K, T) in enumerate(shapes)]
    lead = mppi.Planner(insts[0]["params"], lanes=16)
    pls = [lead] + [mppi.Planner(s["params"], lanes=16, hip_stream=lead.stream()) for s in insts[1:]]
    print("  case:", shapes, asked, flush=True)
    try:
        for i, occ in asked.items():
            pls[i].set_occupancy(occ)
        mppi.step_batch(pls, np.array([s["x0"] for s in insts]),
                        [(s["waypoints"], s["circles"]) for s in insts])
        got = [pl.kernel() for pl in pls]
        # (k_batch's compilation is the tuning table's unless one is asked for)
        assert [SPLIT if k == SPLIT else asked.get(i, 0) for i, k in enumerate(got)] == kernels
        assert all(got[i] == occ for i, occ in asked.items())
        for pl, s in zip(pls, insts):
            with mppi.Planner(s["params"], lanes=16) as ref:
                ref.step(s["x0"], s["waypoints"], s["circles"])
                assert np.array_equal(pl.costs(), ref.costs())
                assert np.array_equal(pl.controls(), ref.controls())
    finally:
        for pl in reversed(pls):
            pl.close()
