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


# (dt, circle speed, radius, step at which it is near, x where it starts): late in
# long horizons, where the times of steps are coarse in float32, and circles whose
# radius is
@pytest.mark.parametrize("dt,v,radius,step,x", [
    (0.291, 29670.8, 1.0, 1920, -16586301.0), (0.258, 25993.1, 1.0, 1984, -13311842.0),
    (0.408, 28912.8, 1.0, 1311, -15476910.0), (0.274, 1528.4, 1.0, 1952, -817876.9375),
    (0.283, 1264.3, 1.0, 1951, -698423.0625), (0.283, 1136.2, 1.0, 1823, -586500.8125),
    (0.271, 1.9, 2979922.0, 1024, 2979396.5), (0.466, 1.8, 2381847.0, 879, -2382587.5),
    (0.074, 6.0, 2887852.0, 176, 2887775.75), (0.076, 48.0, 3121625.0, 831, -3124662.5)])
@pytest.mark.parametrize("n_c", [1, 70])
def test_circles_at_the_resolution_of_float32(dt, v, radius, step, x, n_c):
    """A circle that comes just within the safety distance of a standing vehicle
    at the first or last step of a span of 16 counts as it does in the full
    scan, listed and in a group."""
    mppi = _mppi()
    T = 16 * (step // 16 + 1)
    p = dict(scenes.params(K=1, T=T, dt=dt, v_max=1.0, seed=1), sigma=(0.0, 0.0), ego_off=(0.0,),
             ego_r=0.5, d_safe_c=0.0, d_safe_0=2.0, w_track=0.0, w_speed=0.0, w_effort=0.0, w_coll=1.0)
    wp = np.zeros((3, 4))
    wp[:, 0] = np.arange(3.0)
    ci = np.zeros((n_c, 5))
    ci[:, 0], ci[:, 2] = 1e7, 1.0
    ci[n_c // 2] = x, 0.0, radius, v, 0.0
    _say(dt, v, radius, step, x, n_c)
    got = []
    for cull, occ in ((False, -1), (True, -1), (True, 0)):
        with mppi.Planner(p, lanes=8) as pl:
            pl.set_culling(cull)
            pl.set_occupancy(occ)
            pl.step(np.zeros(4), wp, ci)
            got.append(pl.costs()[0])
    assert got[0] > 0.0
    assert got[1] == got[0] and got[2] == got[0], got
