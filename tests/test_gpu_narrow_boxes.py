"""The launch of boxes at most 32 cells wide: 32 threads along x on two queues
in four- and eight-byte storage, 64 in the one-queue step and in two-byte
storage; the same results with either."""
import math

import numpy as np
import pytest

from iblb_inputs import mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [0, 1, 2, 3])
@pytest.mark.parametrize("nx,drops", [(32, 260), (27, 260), (32, 5)])
def test_default_launch_of_narrow_boxes(nx, drops, storage):
    import paper_2604_17463_amd as P
    say("narrow boxes", nx, drops, storage)
    rng = np.random.default_rng(8)
    ds = []
    for _ in range(drops):  # one node block each; more than 256 take two queues
        v, t = mesh.sphere(0, 2.0, rng.uniform((0, 0, 4), (nx, 64, 60)))
        ds.append(Droplet(0, v, t, sigma=0.004, theta_eq=math.pi, xi=0.3, k_vol=0.0))
    wl = Workload("narrow", [Box(nx, 64, 64, tau=0.9)], ds, storage=storage)
    out = []
    for launch in (None, (64, 2, 1, 0, 0, 0)):
        s = P.Simulation(wl, storage=storage, flags=1, dev_scale=4096.0 if storage == 2 else 1.0)
        if launch:
            s.set_launch(*launch)
        else:
            narrow = drops > 256 and storage < 2
            assert s.get_launch()[:3] == ((32, 8, 1) if narrow else (64, 4, 1))
        s.step(5)
        out.append([s.read_state(0), s.read_nodes(drops - 1)])
        s.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
