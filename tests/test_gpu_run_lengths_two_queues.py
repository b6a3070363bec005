"""Runs of every graph length on two queues with the band kernel beside the
bulk kernel, from rest and from a pending advection, replayed against eager
steps and against one step at a time, bit for bit.  The launch has to differ
from the default one, with which a context of this size runs on one queue."""
import math

import numpy as np
import pytest

from iblb_inputs import mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import say

pytestmark = pytest.mark.gpu

GRAPH = 1
LAUNCH = (64, 2, 1, 0, 0, 0)


@pytest.mark.parametrize("tau_in", [0.0, 1.4])
@pytest.mark.parametrize("k_vol", [0.0, 2e-3])
def test_runs_on_two_queues_equal_eager_steps(k_vol, tau_in):
    import paper_2604_17463_amd as P
    say("run lengths on two queues", k_vol, tau_in)
    v, t = mesh.sphere_above_wall(3, 8.0, 20.3, 17.6, 0.4)
    wl = Workload("runs", [Box(40, 36, 28, tau=0.8, tau_in=tau_in)],
                  [Droplet(0, v, t, sigma=0.01, theta_eq=math.radians(70), xi=0.4, k_vol=k_vol)], storage=1)

    def run(flags, one_by_one=False):
        s = P.Simulation(wl, storage=1, flags=flags)
        assert s.get_launch() != LAUNCH
        s.set_launch(*LAUNCH)
        out = []
        for n in (2, 4, 8, 16, 32, 1, 8, 16, 21, 67, 40):
            for m in [1] * n if one_by_one else [n]:
                s.step(m)
            # the positions are read between most runs, so that the next one starts from rest
            if n != 21:
                out.append(s.read_nodes(0))
        out.append(s.read_state(0))
        s.close()
        return out

    want = run(0)
    for got in (run(GRAPH), run(GRAPH, one_by_one=True)):
        for a, b in zip(got, want):
            assert np.array_equal(a, b)
