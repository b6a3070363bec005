"""Runs of every graph length, from rest and from a pending advection, replayed
against eager steps, bit for bit, on one queue and in both schedules on two."""
import math

import numpy as np
import pytest

from iblb_inputs import mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import say

pytestmark = pytest.mark.gpu

GRAPH = 1


@pytest.mark.parametrize("launch", [None, (64, 4, 1, 0, 0, 0), (64, 2, 1, 0, 0, 1)])
@pytest.mark.parametrize("k_vol", [0.0, 2e-3])
def test_runs_from_rest_equal_eager_steps(launch, k_vol):
    import paper_2604_17463_amd as P
    say("run lengths", launch, k_vol)
    v, t = mesh.sphere_above_wall(3, 8.0, 20.3, 17.6, 0.4)
    wl = Workload("runs", [Box(40, 36, 28, tau=0.8)],
                  [Droplet(0, v, t, sigma=0.01, theta_eq=math.radians(70), xi=0.4, k_vol=k_vol)], storage=1)

    def run(flags):
        s = P.Simulation(wl, storage=1, flags=flags)
        if launch:
            s.set_launch(*launch)
        out = []
        for n in (2, 4, 8, 16, 32, 1, 21, 67):
            s.step(n)
            # the positions are read between most runs, so that the next one starts from rest
            if n != 21:
                out.append(s.read_nodes(0))
        out.append(s.read_state(0))
        s.close()
        return out

    for a, b in zip(run(GRAPH), run(0)):
        assert np.array_equal(a, b)
