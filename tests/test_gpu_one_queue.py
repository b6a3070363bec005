"""The one-queue step of small contexts (fused launches) against the two-queue
schedules, bit for bit: rows shorter and longer than a workgroup, padded and
not, walls at rest and moving, periodic z, with and without a volume penalty
and a viscosity contrast, several boxes with and without droplets, graphs and
eager launches, runs of every graph length."""
import math

import numpy as np
import pytest

from iblb_inputs import mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import say

pytestmark = pytest.mark.gpu

GRAPH, FULL_U = 1, 4


def _drop(box, level, r, c, k_vol=0.0, theta=70.0):
    v, t = mesh.sphere(level, r, c)
    return Droplet(box, v, t, sigma=0.01, theta_eq=math.radians(theta), xi=0.3, k_vol=k_vol)


CASES = {
    "padded": lambda: ([Box(45, 37, 24, tau=0.8)], [_drop(0, 3, 8.0, (22.2, 18.1, 8.7), 2e-3)]),
    "narrow": lambda: ([Box(9, 30, 30, tau=0.7, zbc=1, body_force=(1e-6, 0, 2e-6))],
                       [_drop(0, 2, 3.5, (4.1, 29.2, 27.8), theta=180.0)]),
    "segments": lambda: ([Box(301, 14, 12, tau=0.9)], [_drop(0, 2, 4.0, (299.2, 7.0, 5.0), 1e-3)]),
    "moving": lambda: ([Box(40, 24, 20, tau=1.0, wall_lo=(-0.01, 0.003), wall_hi=(0.01, 0.0))],
                       [_drop(0, 3, 6.0, (20, 12, 10), theta=180.0)]),
    "contrast": lambda: ([Box(40, 32, 70, tau=1.0, tau_in=1.6)], [_drop(0, 3, 7.0, (39.3, 16.2, 30.4))]),
    "contrast_penalty": lambda: ([Box(36, 32, 24, tau=1.0, tau_in=0.7)], [_drop(0, 3, 7.0, (18.3, 16.2, 9.4), 1e-3)]),
    "large": lambda: ([Box(125, 120, 68, tau=0.8)], [_drop(0, 5, 22.0, (60.2, 61.1, 22.7), 2e-3)]),
    "large_contrast": lambda: ([Box(90, 80, 70, tau=1.0, tau_in=1.6)], [_drop(0, 4, 16.0, (85.3, 40.2, 30.4))]),
    "boxes": lambda: ([Box(32, 24, 20, tau=0.8), Box(20, 12, 16, tau=0.9), Box(70, 20, 24, tau=0.7, zbc=1)],
                      [_drop(0, 3, 6.0, (16, 12, 7)), _drop(2, 2, 5.0, (60, 10, 12), 1e-3, 180.0),
                       _drop(2, 1, 3.0, (20, 10, 12), theta=180.0)]),
}


@pytest.mark.parametrize("storage", [0, 1, 2, 3])
@pytest.mark.parametrize("name", sorted(CASES))
def test_one_queue_steps_equal_the_two_queue_schedules(name, storage):
    import paper_2604_17463_amd as P
    say("one queue", name, storage)
    boxes, drops = CASES[name]()
    wl = Workload(name, boxes, drops, storage=storage)
    scale = 4096.0 if storage == 2 else 1.0

    def run(flags, launch, lengths):
        s = P.Simulation(wl, storage=storage, flags=flags, dev_scale=scale)
        if launch:
            s.set_launch(*launch)
        for n in lengths:
            s.step(n)
        out = [s.read_state(b, want_u=True) for b in range(len(boxes))], [s.read_nodes(d) for d in range(len(drops))]
        _, obs = s.observables()
        assert all(b["status_bits"] == 0 for b in obs)
        return out

    full = FULL_U if name == "boxes" else 0
    want = run(full, (64, 2, 1, 0, 0, 0), (23,))
    got = [run(GRAPH | full, None, (1, 1, 18, 3)), run(full, None, (23,))]
    if "contrast" not in name:
        got.append(run(GRAPH | full, (64, 2, 1, 0, 0, 1), (23,)))
    for states, nodes in got:
        for (f, u), (fw, uw) in zip(states, want[0]):
            assert np.array_equal(f, fw)
            assert np.array_equal(u, uw, equal_nan=True)
        for q, qw in zip(nodes, want[1]):
            assert np.array_equal(q, qw)
