"""bench.py's reading of the iteration timing by launch (CPU)."""
import bench

SIX = dict(yfwd=10.0, zsym=12.0, yinv=9.5, rowinv=9.5, upd=6.0, rowfwd=10.0)


def test_launches_of_equal_duration_are_not_taken_for_one():
    assert bench.launch_ms(SIX, 128, "fp64") == SIX
    assert bench.launch_ms(SIX, 256, "mixed") == SIX
    assert bench.launch_ms(SIX, 128, "mixed") == dict(zsym=12.0, planeinv=19.0, upd=6.0, yfwd=10.0, rowfwd=10.0)


def test_shares_of_one_launch_are_added_up():
    assert bench.launch_ms(SIX, 64, "fp64") == dict(zsym=12.0, planeinv=19.0, upd=6.0, planefwd=20.0)
    assert bench.launch_ms(dict(cols=5.0, rowinv=4.0, upd=4.0, rowfwd=4.0), 512, "fp64") == dict(cols=5.0, rows=12.0)
    four = dict(cols=5.0, rowinv=4.0, upd=3.0, rowfwd=4.0)
    assert bench.launch_ms(four, 4096, "fp64") == four
