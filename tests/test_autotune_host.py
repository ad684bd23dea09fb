"""The tuner's choice of a launch shape from given times (no GPU): lanes by the
kernel that the library launches, the other columns by k_batch."""
import pytest

from paper_2308_01654_amd import autotune


def _tune(monkeypatch, ms, split_at):
    """tune_shape with ms[(lanes, occupancy)] (and 1.1 times that without the LDS
    copy); the library's own choice is the split kernel at split_at, timed as
    occupancy -1, elsewhere k_batch as its old table has it."""
    asked = []

    def time_shape(sc, lanes, reps, rounds=3, stage=1, occ=-1):
        asked.append((lanes, stage, occ))
        kernel = autotune.SPLIT if occ < 0 and lanes in split_at else max(occ, 0)
        return ms[(lanes, occ)] * (1.0 if stage else 1.1), kernel

    monkeypatch.setattr(autotune, "time_shape", time_shape)
    return autotune.tune_shape(None, (2, 8, 16), 5), asked


@pytest.mark.parametrize("split_ms,lanes", [(0.5, 16), (1.5, 2)])
def test_lanes_by_the_kernel_that_is_launched(monkeypatch, split_ms, lanes):
    """16 lanes win with the split kernel's time and lose with k_batch's."""
    ms = {(2, -1): 1.0, (2, 0): 1.0, (8, -1): 9.0, (8, 0): 2.0, (8, 1): 1.9,
          (16, -1): split_ms, (16, 0): 3.0, (16, 1): 2.5}
    (times, best, stage, occ, k_batch), asked = _tune(monkeypatch, ms, {16})
    assert best == lanes
    # 8 lanes: k_batch's faster compilation, whatever the old table took
    assert times == {2: 1.0, 8: 1.9, 16: split_ms}
    # the columns are k_batch's at the chosen lanes
    assert (stage, occ) == (1, 1 if lanes == 16 else 0)
    assert k_batch == ({(1, 0): 3.0, (0, 0): 3.0 * 1.1, (1, 1): 2.5} if lanes == 16
                       else {(1, 0): 1.0, (0, 0): 1.1})
    # below 8 lanes there is no second compilation to ask for
    assert not [a for a in asked if a[0] < 8 and a[2] == 1]


def test_every_time_is_of_a_kernel_that_can_be_launched(monkeypatch):
    """Each number of lanes is timed with the library's own choice first."""
    ms = {(g, o): 1.0 for g in (2, 8, 16) for o in (-1, 0, 1)}
    _, asked = _tune(monkeypatch, ms, {8, 16})
    assert [a for a in asked if a[2] == -1] == [(2, 1, -1), (8, 1, -1), (16, 1, -1)]
