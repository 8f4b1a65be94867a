"""What a context holds after a launch that failed (no GPU needed)."""
import pytest

import hip_stand_in

SCRIPT = r"""
precision, count, dt = sys.argv[2], int(sys.argv[3]), 0.01
for done, steps in ((0, 0), (1, 16), (2, 32)):   # launches that go through, steps they take
    tr = lpt.Tracker(16, precision)
    u = np.zeros((16, 16))
    tr.set_snapshot(0, 0.0, u, u)
    tr.set_snapshot(1, 1.0, u, u)
    x = np.linspace(0.0, 6.0, count)
    tr.add_species("tracer", 0.0, "bilinear", x, x)
    hip.stand_in_fail_after(done)
    try:
        tr.step(40, dt)
        raise SystemExit("the failed launch was not reported")
    except lpt.LptError as e:
        assert e.status == lpt.E_HIP, e
    hip.stand_in_fail_after(-1)
    t = 0.0
    for _ in range(steps):
        t += dt
    assert tr.get_time() == (steps, t), (done, tr.get_time())
    tr.step(40 - steps, dt)   # and goes on from there
    assert tr.get_time()[0] == 40
    tr.close()
print("held")
"""


@pytest.mark.parametrize("count", [100, (1 << 18) + 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
def test_time_stays_at_the_last_enqueued_launch(tmp_path, precision, count):
    assert hip_stand_in.run(SCRIPT, tmp_path, precision, count).strip() == "held"
