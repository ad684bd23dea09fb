"""Inputs that are finite as given but whose distances, speeds or weights leave
the range or the resolution of float32: the culled scans of every iteration
kernel give what the full scans give."""
import numpy as np
import pytest

from paper_2308_01654_amd import scenes

pytestmark = pytest.mark.gpu


def _mppi():
    from paper_2308_01654_amd import mppi
    mppi.load()
    return mppi


def _say(*a):
    print("  case:", *a, flush=True)


# one chunk, a last chunk that is not the 16th, all 64 that a wave's lanes hold,
# and past them; where one waypoint is near, all chunks are scanned and it is found
@pytest.mark.parametrize("n_wp", [1, 70, 512, 700])
@pytest.mark.parametrize("lanes,occ", [(16, -1), (8, -1), (4, -1), (16, 0), (16, 1), (2, -1), (1, -1)])
def test_waypoints_whose_squared_distance_is_beyond_float32(lanes, occ, n_wp):
    """No closest waypoint exists in float32: every cost is non-finite, the step
    reports it and keeps the controls.  With one waypoint at hand the costs are
    those of the full scan."""
    mppi = _mppi()
    sc = scenes.tiny(K=70, T=64, n_c=5, seed=3)
    wp = np.zeros((n_wp, 4))
    wp[:, 0] = np.linspace(1e20, 2e20, n_wp)
    wp[:, 3] = 10.0
    near = wp.copy()
    near[n_wp // 2, :2] = 3.0, 1.0
    for what, w in (("far", wp), ("near", near)):
        outs = []
        for cull in (True, False):
            _say(lanes, occ, n_wp, what, "culling", cull)
            # a capacity of just these waypoints: nothing of the handle's lies behind them
            with mppi.Planner(sc["params"], max_waypoints=n_wp, lanes=lanes) as pl:
                pl.set_occupancy(occ)
                pl.set_culling(cull)
                U = pl.controls()
                pl.step(sc["x0"], w, sc["circles"])
                if what == "far":
                    with pytest.raises(mppi.MppiError) as e:
                        pl.sync()
                    assert e.value.status == mppi.E_NONFINITE
                    assert np.array_equal(pl.get_state()[0], U)
                outs.append(pl.costs())
        assert np.array_equal(outs[0], outs[1], equal_nan=True)
        assert np.all(np.isfinite(outs[0]) == (what == "near"))


# a safety distance that is +inf in float32 for every state, for those in motion
# (0 * inf is not a number for the others), and -inf; a start so fast that
# positions leave float32 along the horizon, and headings before positions do;
# circles listed at once and in groups, one ego circle and four
@pytest.mark.parametrize("n_c", [1, 20, 40, 90, 300])
@pytest.mark.parametrize("name,over", [
    ("distance", dict(d_safe_0=1e39)), ("per speed", dict(d_safe_c=1e39)),
    ("negative", dict(d_safe_0=-1e39)), ("both", dict(d_safe_0=1e39, collision_only=1)),
    ("fast", dict(v_max=1e300)), ("fast, hit", dict(v_max=1e300, collision_only=1)),
    ("heading", dict(v_max=1e300, wheelbase=4e-39)),
    ("four", dict(d_safe_0=1e39, ego_off=(0.0, 1.0, 2.0, 3.0)))])
def test_states_and_safety_distances_beyond_float32(name, over, n_c):
    """Costs of the culled scans, by wave and by rows, equal the full scans'
    where the safety distance, the position or the heading is not finite."""
    mppi = _mppi()
    rng = np.random.Generator(np.random.PCG64(n_c))
    sc = scenes.tiny(K=90, T=70, n_c=0, seed=4)
    p = dict(sc["params"], **over)
    x0 = np.array(sc["x0"])
    if "v_max" in over:
        x0[3] = 3e37 if name != "heading" else 10.0
    ci = scenes.sine_circles(rng, n_c, 0.0, 60.0)
    for lanes in (16, 8, 4):
        outs = []
        for cull, occ in ((0, -1), (1, -1), (1, 0)):
            _say(name, n_c, lanes, "culling", cull, "occupancy", occ)
            with mppi.Planner(p, lanes=lanes) as pl:
                pl.set_occupancy(occ)
                pl.set_culling(cull)
                pl.step(x0, sc["waypoints"], ci)
                outs.append(pl.costs())
        for o in outs[1:]:
            assert np.array_equal(outs[0], o, equal_nan=True), (lanes, outs[0][:4], o[:4])


@pytest.mark.parametrize("lanes", [16, 8, 4])
def test_obstacle_weight_beyond_float32_without_obstacles(lanes):
    """An instance without obstacle circles has no obstacle term whatever its
    weight, alone and in a batch with instances that have circles."""
    mppi = _mppi()
    free = scenes.tiny(K=60, T=70, n_c=0, seed=4)
    free["params"] = dict(free["params"], w_coll=1e39)
    other = scenes.tiny(K=60, T=70, n_c=6, seed=5)
    _say(lanes)
    with mppi.Planner(free["params"], lanes=lanes) as pl:
        pl.step(free["x0"], free["waypoints"], free["circles"])
        alone = pl.costs(), pl.controls()
    assert np.all(np.isfinite(alone[0]))
    with mppi.Planner(free["params"], lanes=lanes) as pl, \
            mppi.Planner(other["params"], lanes=lanes, hip_stream=pl.stream()) as q:
        mppi.step_batch([pl, q], np.array([free["x0"], other["x0"]]),
                        [(s["waypoints"], s["circles"]) for s in (free, other)])
        assert np.array_equal(pl.costs(), alone[0])
        assert np.array_equal(pl.controls(), alone[1])
        q.sync()
