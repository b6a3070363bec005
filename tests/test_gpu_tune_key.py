"""Kept autotune results: configurations whose steps are made of different
launches (a volume penalty or none, as many nodes in more node blocks) are
timed apart."""
import math

import numpy as np
import pytest

from iblb_inputs import mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import say

pytestmark = pytest.mark.gpu

GRAPH, AUTOTUNE = 1, 2


def _workload(freqs, k_vol):
    drops = []
    for k, freq in enumerate(freqs):
        v, t = mesh.geodesic(freq)
        drops.append(Droplet(0, 4.0 * v + np.array((10.0 + 14.0 * k, 12.0, 9.5)), t, sigma=0.01, theta_eq=math.pi,
                             xi=0.3, k_vol=k_vol))
    return Workload("tune-key", [Box(52, 24, 20, tau=0.8)], drops, storage=1)


def test_penalty_and_node_blocks_are_part_of_the_key(tmp_path, monkeypatch):
    import paper_2604_17463_amd as P
    say("tune key")
    path = str(tmp_path / "tune.txt")
    monkeypatch.setenv("IBLB_TUNE_CACHE", path)
    # 162 + 162 + 12 and 252 + 42 + 42 nodes: seven blocks of 64 and six
    a, b = (4, 4, 1), (5, 2, 2)
    assert sum(10 * f * f + 2 for f in a) == sum(10 * f * f + 2 for f in b)
    for n, (freqs, k_vol) in enumerate(((a, 0.0), (a, 1e-3), (b, 0.0))):
        P.Simulation(_workload(freqs, k_vol), storage=1, flags=GRAPH | AUTOTUNE).close()
        keys = {line.split("\t")[0] for line in open(path).read().splitlines()}
        assert len(keys) == n + 1, keys
