"""The particle state is one allocation (no GPU needed): what a context costs to
set up goes by the number of its allocations."""
import pytest

import hip_stand_in

SCRIPT = r"""
tr = lpt.Tracker(16, sys.argv[2])
u = np.zeros((16, 16))
tr.set_snapshot(0, 0.0, u, u)
tr.set_snapshot(1, 1.0, u, u)
for count in (1000, 77):
    x = np.linspace(0.0, 6.0, count)
    hip.stand_in_mallocs()
    tr.add_species("inertial", 0.5, "bilinear", x, x, x, x)
    print(hip.stand_in_mallocs())
"""


@pytest.mark.parametrize("precision", ["fp64", "fp32_split"])
def test_one_allocation_holds_the_state(tmp_path, precision):
    first, second = map(int, hip_stand_in.run(SCRIPT, tmp_path, precision).split())
    # four host arrays staged, the statistics partials and records, and the state
    assert first <= 7 and second <= 7, (first, second)
