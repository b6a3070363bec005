"""The band kernel's two grids: beside the bulk kernel (one workgroup per node
block, more where there are few) each wave takes several tiles of the list;
alone, one wave per tile the box could hold, in eighths of the list.  Both
schedules give the same bits."""
import math

import numpy as np
import pytest

from iblb_inputs import mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", [0, 1, 3])
@pytest.mark.parametrize("level", [0, 2, 5])
def test_band_grids_give_the_same_bits(level, storage):
    # 5 x 65 x 128 = 41,600 tiles: the grid alone is the largest (8,192
    # workgroups); one block of 12 nodes, three of 162, 161 of 10,242
    import paper_2604_17463_amd as P
    say("band grids", level, storage)
    v, t = mesh.sphere(level, 26.0, (147.3, 64.2, 60.1))
    wl = Workload("band-grids", [Box(150, 130, 128, tau=0.8)],
                  [Droplet(0, v, t, sigma=0.01, theta_eq=math.pi, xi=0.3, k_vol=0.0)], storage=storage)

    def run(after):
        s = P.Simulation(wl, storage=storage, flags=1)
        s.set_launch(64, 4, 1, 0, 0, after)
        s.step(7)
        f, u = s.read_state(0, want_u=True)
        q = s.read_nodes(0)
        s.close()
        return f, u, q

    for a, b in zip(run(0), run(1)):
        assert np.array_equal(a, b, equal_nan=True)
