"""Scenes staged while the device is behind, and under the caller's capture."""
import ctypes

import numpy as np
import pytest

from paper_2308_01654_amd import scenes

pytestmark = pytest.mark.gpu


def _mppi():
    from paper_2308_01654_amd import mppi
    mppi.load()
    return mppi


def _hip():
    from paper_2308_01654_amd.hip_events import HipEvents
    return HipEvents().H


def _ok(status):
    assert status == 0, status


def _scenes(n, **kw):
    """The same planner in n different scenes."""
    out = []
    for i in range(n):
        sc = scenes.tiny(seed=20 + i, **kw)
        sc["params"] = dict(sc["params"], seed=1)
        out.append(sc)
    return out


def _capture(hip, stream, calls):
    graph, run = ctypes.c_void_p(), ctypes.c_void_p()
    _ok(hip.hipStreamBeginCapture(stream, 1))  # thread local
    calls()
    _ok(hip.hipStreamEndCapture(stream, ctypes.byref(graph)))
    _ok(hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)))
    _ok(hip.hipGraphDestroy(graph))
    return run


def test_long_steps_enqueued_without_a_read():
    """Steps of several times the time that the host looks for a free staging
    buffer, each in a scene of its own: the controls of steps with a read after
    each."""
    mppi = _mppi()
    scs = _scenes(7, K=262144, T=100, n_c=40)
    got = []
    for read in (True, False):
        with mppi.Planner(scs[0]["params"]) as pl:
            for sc in scs:
                pl.step(sc["x0"], sc["waypoints"], sc["circles"])
                if read:
                    pl.sync()
            got.append(pl.controls())
    assert np.array_equal(*got)


def test_step_captured_behind_queued_work():
    """A step is captured while both staging buffers of its handle wait behind
    milliseconds of another's work on the stream; its graph does what steps do."""
    mppi, hip = _mppi(), _hip()
    scs = _scenes(3, K=300, T=20, n_c=3)
    long = _scenes(1, K=262144, T=100, n_c=40)[0]
    with mppi.Planner(long["params"]) as slow, \
            mppi.Planner(scs[0]["params"], hip_stream=slow.stream()) as pl, \
            mppi.Planner(scs[0]["params"]) as alone:
        stream = ctypes.c_void_p(slow.stream())
        slow.step(long["x0"], long["waypoints"], long["circles"])
        slow.sync()
        for _ in range(8):
            slow.step_resident(long["x0"])
        for sc in scs[:2]:
            pl.step(sc["x0"], sc["waypoints"], sc["circles"])
        run = _capture(hip, stream, lambda: pl.step(scs[2]["x0"], scs[2]["waypoints"], scs[2]["circles"]))
        for _ in range(3):
            _ok(hip.hipGraphLaunch(run, stream))
        for sc in scs[:2] + 3 * scs[2:]:
            alone.step(sc["x0"], sc["waypoints"], sc["circles"])
        assert np.array_equal(pl.controls(), alone.controls())
        assert pl.get_state()[1] == alone.get_state()[1] == 5
        _ok(hip.hipGraphExecDestroy(run))


def test_two_scenes_of_a_handle_in_one_capture():
    """Two scenes can be captured together, a third is refused without harm to the
    capture or the handle; scenes staged between launches of the graph are read
    as given."""
    mppi, hip = _mppi(), _hip()
    scs = _scenes(4, K=300, T=20, n_c=3)
    with mppi.Planner(scs[0]["params"]) as pl, mppi.Planner(scs[0]["params"]) as alone:
        stream = ctypes.c_void_p(pl.stream())

        def step(q, i):
            q.step(scs[i]["x0"], scs[i]["waypoints"], scs[i]["circles"])

        def calls():
            step(pl, 0)
            step(pl, 1)
            with pytest.raises(mppi.MppiError) as e:
                step(pl, 2)
            assert e.value.status == mppi.E_INVALID

        run = _capture(hip, stream, calls)
        for _ in range(2):
            _ok(hip.hipGraphLaunch(run, stream))
            for i in (0, 1):
                step(alone, i)
        assert np.array_equal(pl.controls(), alone.controls())
        # scenes of the caller's own turn, after launches that have ended
        for _ in range(2):
            for i in (2, 3, 2):
                step(pl, i)
                step(alone, i)
            assert np.array_equal(pl.controls(), alone.controls())
        _ok(hip.hipGraphExecDestroy(run))
