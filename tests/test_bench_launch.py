"""The benchmark's figure for the launch by itself is one of the shape that
the timed loop ran, and names the shape it timed.  CPU only."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench


class Tuner:
    """A context whose autotuner picks these shapes in turn."""

    def __init__(self, picks):
        self.picks, self.calls = list(picks), []

    def set_params(self, table_mode, tiles_per_wg, autotune):
        self.calls.append((table_mode, tiles_per_wg, autotune))
        self.now = self.picks.pop(0)

    def tiling(self):
        return [self.now]


def shape(resident, tpw, split):
    return {"resident": resident, "tpw": tpw, "split": split, "JC": 3}


def test_the_pick_is_repeated_until_it_is_the_timed_one():
    c = Tuner([shape(1, 4, 0), shape(0, 2, 4), shape(0, 1, 4)])
    got = bench.launch_alone(c, shape(0, 1, 4), c.set_params, tuned=True)
    assert got == shape(0, 1, 4) and c.calls == [("auto", 0, True)] * 3


def test_another_pick_is_returned_as_what_it_is():
    c = Tuner([shape(1, 4, 0)] * 5)
    got = bench.launch_alone(c, shape(0, 1, 3), c.set_params, tuned=True)
    assert bench.tables_of(got) == "resident" and len(c.calls) == 5


def test_named_shapes_are_forced_and_untimed_ones_stay_untimed():
    c = Tuner([shape(1, 2, 0)])
    assert bench.launch_alone(c, shape(1, 2, 0), c.set_params, tuned=True) == shape(1, 2, 0)
    assert c.calls == [("resident", 2, False)]
    c = Tuner([shape(0, 1, 3)])
    assert bench.launch_alone(c, shape(0, 1, 3), c.set_params, tuned=False) == shape(0, 1, 3)
    assert c.calls == [("auto", 0, False)]
