"""Timing the mesh chain leaves the run unchanged where the tiles record their
node blocks (a box of more than 256 blocks): the step after it must not meet
the records of the last repetition."""
import math

import numpy as np
import pytest

from iblb_inputs import mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reps", [1, 4])
@pytest.mark.parametrize("storage", [0, 1])
def test_timing_the_mesh_chain_of_many_blocks(storage, reps):
    import paper_2604_17463_amd as P
    say("mesh chain timing, many blocks", storage, reps)
    rng = np.random.default_rng(5)
    drops = []
    for _ in range(300):  # one block each
        v, t = mesh.sphere(0, 2.0, rng.uniform((0, 0, 4), (64, 56, 36)))
        drops.append(Droplet(0, v, t, sigma=0.004, theta_eq=math.pi, xi=0.3, k_vol=0.0))
    wl = Workload("many-blocks", [Box(64, 56, 40, tau=0.9)], drops, storage=storage)

    def run(timed):
        s = P.Simulation(wl, storage=storage, flags=1)
        for n in (0, 1, 3):
            s.step(n)
            if timed:
                assert s.time_mesh_chain(reps=reps) > 0.0
        s.step(1)
        _, obs = s.observables()
        assert obs[0]["status_bits"] == 0
        out = [s.read_state(0)] + [s.read_nodes(d) for d in range(len(drops))]
        s.close()
        return out

    for a, b in zip(run(True), run(False)):
        assert np.array_equal(a, b)
