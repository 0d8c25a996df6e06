"""The batch tuner also times the library's own choice where that is one no
explicit execution names (narrow, periodic chambers without space charge), and
keeps it if it is the fastest."""
import time

import pytest

from test_autotune_host import _batch, tuner  # noqa: F401


@pytest.mark.parametrize("over,tried", [({}, True), (dict(n_pulses=3, pulse_period_s=2e-8), True),
                                        (dict(lateral_bc=1), False), (dict(space_charge=1), False),
                                        (dict(nx=64, ny=33), False)])
def test_the_librarys_choice_is_timed(tuner, monkeypatch, over, tried):  # noqa: F811
    calls = []

    def run(chs, trs, exec=None, ws=None, stream=None):
        calls.append(dict(exec))
        time.sleep(0.0 if exec["kernel"] == tuner.B.IT_KERNEL_AUTO else 0.005)
        return [dict(f=1.0, ks=1.0, flags=0) for _ in chs]
    monkeypatch.setattr(tuner.B, "it_solve_batch", run)
    chs, trs = _batch(**over)
    ex = tuner.tune_batch(chs, trs, steps=4)
    assert any(c["kernel"] == tuner.B.IT_KERNEL_AUTO for c in calls) == tried
    assert (ex["kernel"] == tuner.B.IT_KERNEL_AUTO) == tried


def test_three_steps_are_timed_with_both_rows(tuner):  # noqa: F811
    rows = {c.get("tile_y") for c in tuner.BLOCKED if c["steps_per_pass"] == 3}
    assert {24, 32} <= rows
