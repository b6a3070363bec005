"""The spread force adds a cell's node blocks in one order whatever launch
takes the step.  Where a block's partial region does not fit, its nodes are
added one by one after the other blocks of its batch, so the batches must not
depend on how many blocks a launch tests at a time: 140 droplets of one block
each, some without a region, close enough that most band tiles meet blocks of
several groups of 64."""
import math

import numpy as np
import pytest

from iblb_inputs import mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import say

pytestmark = pytest.mark.gpu

GRAPH = 1
BIG = (3, 10, 66, 100, 139)  # droplets whose region does not fit


def _cells(q):
    b = np.floor(q - 0.5)
    return int(np.prod(b.max(axis=0) - b.min(axis=0) + 4))


def _workload(storage):
    rng = np.random.default_rng(20)
    drops = []
    for k in range(140):
        r = 5.8 if k in BIG else 2.0
        c = rng.uniform((0, 0, 8), (48, 40, 32))
        v, t = mesh.sphere(1 if k in BIG else 0, r, c)
        assert len(v) <= 64  # one block
        # the limit is 3,200 cells in FP32 and 2,944 in FP64
        assert (_cells(v) > 3200) == (k in BIG) and (k in BIG or _cells(v) < 2944)
        drops.append(Droplet(0, v, t, sigma=0.004, theta_eq=math.pi, xi=0.3, k_vol=1e-3 if k % 2 else 0.0))
    return Workload("sum-order", [Box(48, 40, 40, tau=0.9)], drops, storage=storage)


@pytest.mark.parametrize("storage", [0, 1, 2])
def test_steps_do_not_depend_on_the_launch(storage):
    import paper_2604_17463_amd as P
    say("sum order", storage)
    wl = _workload(storage)

    def run(launch=None, static=False, flags=GRAPH):
        s = P.Simulation(wl, storage=storage, flags=flags, dev_scale=4096.0 if storage == 2 else 1.0)
        if launch:
            s.set_launch(*launch)
        (s.step_static if static else s.step)(4)
        _, obs = s.observables()
        assert obs[0]["status_bits"] == 0
        f, u = s.read_state(0, want_u=True)
        q = np.concatenate([s.read_nodes(d) for d in range(len(wl.droplets))])
        s.close()
        return f, u, q

    want = run()
    for other in (run(flags=0), run((64, 2, 1, 0, 0, 0)), run((64, 2, 1, 0, 0, 1)), run(static=True)):
        for a, b in zip(other, want):
            assert np.array_equal(a, b, equal_nan=True)
