"""The bench's side legs stay within its time budget, so that its one line comes out."""
import bench


def test_legs_past_the_budget_are_left_out():
    now = [0.0]
    b = bench.Budget(540.0, clock=lambda: now[0])
    assert b.fits("a", 165)
    now[0] = 375.0
    assert b.fits("b", 165) and not b.fits("c", 165.5)
    now[0] = 600.0
    assert not b.fits("d", 1)
    assert b.skipped == ["c", "d"]
    b = bench.Budget(0.0, clock=lambda: 1e6)
    assert b.fits("e", 1e6) and b.skipped == []
