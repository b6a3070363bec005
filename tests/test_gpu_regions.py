"""Partial-spread regions of few node blocks: larger than those of many blocks
(2,048 cells), up to what the kernel's LDS holds.  A one-block droplet alone
against the same droplet next to a box of 641 blocks, where its region does
not fit and its nodes are summed one by one: equal up to the order of at most
42 additions per cell and step."""
import math

import numpy as np
import pytest

from iblb_inputs import mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import say

pytestmark = pytest.mark.gpu

F64, F32 = 0, 1
STEPS = 3


def _cells(q):
    b = np.floor(q - 0.5)
    return int(np.prod(b.max(axis=0) - b.min(axis=0) + 4))


# 3,150 cells exceed the FP64 region of 2,944 and fit the FP32 one of 3,200;
# all take two LDS copies in FP32 and one in FP64
@pytest.mark.parametrize("storage", [F64, F32])
@pytest.mark.parametrize("r,y,cells", [(4.6, 19.5, 2197), (5.0, 19.5, 2744), (5.1, 20.0, 3150)])
def test_regions_of_few_blocks(r, y, cells, storage):
    import paper_2604_17463_amd as P
    say("regions", r, storage)
    v, t = mesh.sphere(1, r, (20.5, y, 12.5))
    assert _cells(v) == cells
    v2, t2 = mesh.sphere_above_wall(6, 8.0, 16.4, 18.1, 0.4)
    box, drop = Box(40, 40, 26, tau=0.9), dict(sigma=0.01, theta_eq=math.radians(70), xi=0.25, k_vol=2e-3)

    def run(boxes, drops):
        s = P.Simulation(Workload("regions", boxes, drops, storage=storage), storage=storage, flags=1)
        s.step(STEPS)
        f, u = s.read_state(0, want_u=True)
        q = s.read_nodes(0)
        s.close()
        return f, q - v

    one = run([box], [Droplet(0, v, t, **drop)])
    two = run([box, Box(32, 36, 24, tau=0.8)],
              [Droplet(0, v, t, **drop), Droplet(1, v2, t2, sigma=0.01, theta_eq=math.radians(60), xi=0.4, k_vol=0.0)])
    eps = 2.0 ** -53 if storage == F64 else 2.0 ** -24
    for a, b in zip(one, two):
        scale = np.abs(b).max()
        assert scale > 0
        # positions are read as sums of two parts, so their moves carry the
        # positions' own rounding as well
        assert np.abs(a - b).max() <= 42 * STEPS * eps * scale + 4 * eps * 40 * (a is one[1])
