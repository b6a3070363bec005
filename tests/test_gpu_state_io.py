"""Populations and node positions in and out through the staging chunks of
131,072 values: fields of several chunks with a partial last one, windows that
cross the periodic sides, walls at rest and moving, every storage; each value
bit for bit what the storage's rounding gives."""
import numpy as np
import pytest

from iblb_inputs import configs, mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import say

pytestmark = pytest.mark.gpu

CHUNK = 1 << 17


def _rounded(v, storage, scale):
    if storage == 0:
        return v
    if storage == 1:
        return v.astype(np.float32).astype(np.float64)
    if storage == 2:
        return (v * scale).astype(np.float32).astype(np.float16).astype(np.float64) / scale
    b = v.astype(np.float32).view(np.uint32).astype(np.uint64)
    b = (b + 0x7FFF + ((b >> 16) & 1)) >> 16 << 16
    return b.astype(np.uint32).view(np.float32).astype(np.float64)


@pytest.mark.parametrize("zbc,walls", [(1, ((0.0, 0.0), (0.0, 0.0))), (0, ((0.0, 0.0), (0.0, 0.0))),
                                       (0, ((0.03, -0.02), (-0.01, 0.04)))])
@pytest.mark.parametrize("storage,scale", [(0, 1.0), (1, 1.0), (2, 4096.0), (3, 1.0)])
def test_fields_round_trip_bit_for_bit(storage, scale, zbc, walls):
    import paper_2604_17463_amd as P
    say("fields", storage, zbc, walls)
    nx, ny, nz, rho0 = 61, 23, 17, 1.25
    wl = Workload("io", [Box(8, 8, 8, tau=0.8), Box(nx, ny, nz, tau=0.8, rho0=rho0, zbc=zbc, wall_lo=walls[0],
                                                    wall_hi=walls[1])], [], storage=storage)
    s = P.Simulation(wl, storage=storage, dev_scale=scale)
    c, w = P.velocity_set()
    rest = (w * rho0)[:, None, None, None]
    f = rest * (1.0 + configs.perturbed_populations(wl.boxes[1], 5, 0.05))
    assert f.size > 2 * CHUNK and f.size % CHUNK
    s.write_state(f, 1)
    kick = np.zeros_like(f)  # the moving-wall part of a population reflected at a wall
    if zbc == 0:
        for i in range(19):
            for cz, z, u in ((1, 0, walls[0]), (-1, nz - 1, walls[1])):
                if c[i, 2] == cz:
                    kick[i, z] = 6.0 * w[i] * rho0 * (c[i, 0] * u[0] + c[i, 1] * u[1])
    want = rest + (_rounded((f - kick) - rest, storage, scale) + kick)
    got = s.read_state(1)
    assert np.array_equal(got, want)
    for lo, ext in (((0, 0, 0), (1, 1, 1)), ((nx - 3, ny - 2, 4), (nx, ny, 7)), ((5, 20, 0), (11, 9, nz))):
        ix, iy, iz = [(np.arange(lo[a], lo[a] + ext[a])) % n for a, n in enumerate((nx, ny, nz))]
        assert np.array_equal(s.read_window(lo, ext, 1), want[:, iz[:, None, None], iy[:, None], ix])
    # a value that is not finite, in the last chunk: refused, state as it was
    bad = f * 1.5
    bad[18, -1, -1, -1] = np.inf
    with pytest.raises(P.IblbError) as e:
        s.write_state(bad, 1)
    assert e.value.code == P.IBLB_E_INVAL
    assert np.array_equal(s.read_state(1), want)
    # stepping goes on from the written state whatever buffer it lies in
    t = P.Simulation(wl, storage=storage, dev_scale=scale)
    t.step(1)
    t.write_state(f, 1)
    s.step(3)
    t.step(3)
    assert np.array_equal(s.read_state(1), t.read_state(1))


@pytest.mark.parametrize("storage", [0, 1])
def test_nodes_come_back_in_the_callers_order(storage):
    import paper_2604_17463_amd as P
    say("nodes", storage)
    v, t = mesh.geodesic(67)
    small, ts = mesh.sphere(2, 5.0, (10.0, 9.0, 8.0))
    big = v * 20.0 + np.array([32.3, 31.9, 30.1])
    assert big.size > CHUNK and big.size % CHUNK
    drops = [Droplet(1, big, t, sigma=0.0, theta_eq=1.0, xi=1.0), Droplet(0, small, ts, sigma=0.0, theta_eq=1.0, xi=1.0)]
    wl = Workload("nodes", [Box(20, 20, 20, tau=0.8), Box(64, 64, 64, tau=0.8)], drops, storage=storage)
    s = P.Simulation(wl, storage=storage)
    for d, q in ((0, big), (1, small)):
        hi = q.astype(np.float32).astype(np.float64)
        want = q if storage == 0 else hi + (q - hi).astype(np.float32)
        assert np.array_equal(s.read_nodes(d), want)
