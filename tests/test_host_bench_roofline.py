"""The benchmark's Sign roofline: the operations counted and the time they are divided by cover the same work.
In rounds the loop's events leave out the first round's masks, so the whole call is counted over the whole
call's time; only the loop kernel has its iterations alone between its events."""
import numpy as np
import pytest

import bench


@pytest.mark.parametrize("level", [2, 65])
def test_counted_work_and_window(level):
    lens, its = np.full(1000, 32), 4300
    whole, loop = bench.sign_work(level, lens, its), its * bench.sign_iteration_ops(level)
    assert bench.sign_achieved(level, lens, its, 2.0) == (whole, whole / 2e-3)
    assert bench.sign_achieved(level, lens, its, 2.0, 1.5) == (loop, loop / 1.5e-3)


def test_settings_that_run_in_rounds():
    assert bench.in_rounds(0, "") and bench.in_rounds(4, "") and bench.in_rounds(4, "4,0,0")
    assert not bench.in_rounds(2, "") and not bench.in_rounds(1, "1,0,0")
    assert not bench.in_rounds(4, "4,16,512") and not bench.in_rounds(4, "4,0,512")
