"""Observables at the edges of their partitions: boxes of one row group and of
several, rows not a multiple of a workgroup's four waves, rows of one cell and
past 64; meshes of one triangle chunk (256), of one and a bit and of many;
several droplets and boxes with and without droplets in one context."""
import numpy as np
import pytest

import oracle
from iblb_inputs import configs, mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import lib_to_oracle_perm, say, to_oracle

pytestmark = pytest.mark.gpu

# FP64 sums of at most 1e6 terms in a tree: log2(1e6) ulp of the sum of
# magnitudes; the stored values themselves are read exactly.
TOL = 1e-13


def _drop(box, level, r, c, seed):
    v, t = mesh.sphere(level, r, c)
    v = v + configs.jitter_nodes(np.zeros_like(v), seed, 0.02 * r)
    return Droplet(box, v, t, sigma=0.01, theta_eq=1.2, xi=0.3 * r)


def _workload():
    boxes = [Box(20, 17, 16, tau=0.9), Box(1, 5, 3, tau=0.8), Box(131, 7, 9, tau=0.7, rho0=1.5),
             Box(66, 40, 36, tau=1.1, zbc=1), Box(24, 24, 24, tau=1.0, wall_lo=(0.02, -0.01), wall_hi=(-0.03, 0.01))]
    drops = [_drop(3, 4, 9.0, (20.0, 20.0, 18.0), 1), _drop(0, 1, 4.0, (10.0, 8.5, 8.0), 2),
             _drop(3, 2, 5.0, (50.0, 20.0, 18.0), 3), _drop(4, 3, 7.0, (12.0, 12.0, 12.0), 4)]
    return Workload("edges", boxes, drops, storage=0)


@pytest.mark.parametrize("storage,scale", [(0, 1.0), (1, 1.0), (2, 4096.0), (3, 1.0)])
def test_observables_at_partition_edges(storage, scale):
    import paper_2604_17463_amd as P
    say("observables", storage)
    wl = _workload()
    s = P.Simulation(wl, storage=storage, dev_scale=scale)
    perm = lib_to_oracle_perm()
    _, w, _ = oracle.lattice()
    want = []
    for b, bx in enumerate(wl.boxes):
        f = (w * bx.rho0)[:, None, None, None] * (1.0 + configs.perturbed_populations(bx, 30 + b, 3e-3))
        inv = np.empty_like(f)
        inv[:] = f[perm]
        s.write_state(np.ascontiguousarray(inv), b)
        held = to_oracle(s.read_state(b), perm)
        want.append((held.sum(), oracle.max_u(held)))
    drops, boxes = s.observables()
    for b, (m, u) in enumerate(want):
        assert abs(boxes[b]["mass"] - m) < TOL * m, b
        # rho and j are differences of populations near w: 1e-16 / |j|; the
        # wall term of a moving wall is added in the storage's arithmetic
        assert abs(boxes[b]["max_u"] - u) < (1e-11 if storage == 0 else 2e-6) * u, b
    for d, dr in enumerate(wl.droplets):
        q = s.read_nodes(d)
        o, dfm = oracle.mesh_observables(dr.tris, q, dr.xi), oracle.deformation(dr.tris, q)
        g = drops[d]
        assert g["z_min"] == o["z_min"] and g["z_max"] == o["z_max"] and g["n_crossings"] == o["n_crossings"]
        for k in ("volume", "area", "cx", "cy", "cz", "contact_radius", "theta_app"):
            assert abs(g[k] - o[k]) < 20 * TOL * abs(o[k]), (d, k)
        # D is a difference of eigenvalues near r^2 / 5, of size 2 D r^2 / 5
        assert abs(g["deformation"] - dfm["D"]) < 20 * TOL, d
