"""The largest velocity of a box whose cells leave the range in which squares
of FP64 values can be compared: two such cells of one thread of the sum, the
faster one second."""
import numpy as np
import pytest

from iblb_inputs.configs import Box, Workload

from _helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 1e60, 1e80, 1e150])
def test_largest_velocity_of_extreme_populations(scale):
    import paper_2604_17463_amd as P
    say("extreme populations", scale)
    s = P.Simulation(Workload("fast", [Box(8, 8, 8, tau=1.0, zbc=1)], [], storage=0), storage=0)
    c, w = P.velocity_set()
    f = np.empty((19, 8, 8, 8))
    f[:] = np.asarray(w)[:, None, None, None]
    i = [tuple(v) for v in c].index((1, 0, 0))
    # rows 8 and 12, read by the same threads: velocity 1/2, then 1
    for y, rest in ((0, scale), (4, 0.0)):
        f[:, 1, y, 2] = 0.0
        f[0, 1, y, 2] = rest
        f[i, 1, y, 2] = scale
    s.write_state(f)
    _, obs = s.observables(raise_unstable=False)
    s.close()
    # the stored deviations carry a rounding error of 2^-53 each
    assert obs[0]["max_u"] == pytest.approx(1.0, rel=1e-14)
