"""The sound-speed bit is set from a cell's velocity with its whole force.
Rows of the one-queue step that run beside the moving nodes are computed
before the band tiles are known, without the spread force: a band cell whose
velocity exceeds the sound speed only without it must not set the bit, and a
cell of the same speed outside the band, in the droplet's box or in one
without droplets, must."""
import math

import numpy as np
import pytest

import oracle
from iblb_inputs import mesh
from iblb_inputs.configs import Box, Droplet, Workload

from _helpers import lib_to_oracle_perm, say, to_lib

pytestmark = pytest.mark.gpu

MACH = 2
CS = math.sqrt(1.0 / 3.0)
BAND, FREE = (12, 12, 22), (2, 3, 24)  # at the top of the droplet; outside every stencil


def _workload(storage, k_vol, boxes=1):
    v, t = mesh.sphere(3, 6.5, (12.5, 12.5, 15.5))
    drop = Droplet(0, v, t, sigma=0.05, theta_eq=math.pi, xi=0.3, k_vol=k_vol)
    return Workload("mach", [Box(24, 24, 28, tau=5.0) for _ in range(boxes)], [drop], storage=storage)


def _populations(cell, amp):
    """Fluid at rest, but for populations moving up around `cell` that all
    reach it in one step."""
    c, w, _ = oracle.lattice()
    f = np.empty((19, 28, 24, 24))
    f[:] = w[:, None, None, None]
    x, y, z = cell
    for i in range(19):
        if c[i][2] == 1:
            f[i, z - 1, y - c[i][1], x - c[i][0]] += amp
    return f


def _second_step(wl, cell, amp):
    """Bare velocity (no spread force) of step 2 at every cell, the velocity
    with its whole force of steps 1 and 2, and the force density at `cell`
    over twice the density."""
    o = oracle.OracleSim(wl, f0=[_populations(cell, amp)])
    o.step(1)
    u1 = o.last_u[0].copy()
    c, _, _ = oracle.lattice()
    f = o.f[0].copy()
    bare = np.einsum("ia,izyx->azyx", c.astype(float), f) / f.sum(axis=0)
    o.step(1)
    x, y, z = cell
    half = o.last_F[0][2, z, y, x] / (2.0 * f[:, z, y, x].sum())
    return bare, u1, o.last_u[0].copy(), half


def _amplitude(wl, cell, excess):
    """amp for which the bare speed at `cell` in step 2 is the sound speed
    plus excess times the half force that holds it back."""
    lo, hi = 0.0, 2.0
    x, y, z = cell
    for _ in range(60):
        amp = 0.5 * (lo + hi)
        bare, _, _, half = _second_step(wl, cell, amp)
        if np.linalg.norm(bare[:, z, y, x]) < CS + excess * abs(half):
            lo = amp
        else:
            hi = amp
    return amp


def _status(P, wl, storage, fields, launch):
    s = P.Simulation(wl, storage=storage, flags=1)
    if launch:
        s.set_launch(*launch)
    perm = lib_to_oracle_perm()
    for b, f in enumerate(fields):
        if f is not None:
            s.write_state(to_lib(f, perm), b)
    s.step(2)
    _, obs = s.observables(raise_unstable=False)
    s.close()
    return obs[0]["status_bits"]


@pytest.mark.parametrize("launch", [None, (64, 2, 1, 0, 0, 0)])
@pytest.mark.parametrize("k_vol", [0.0, 1e-3])
@pytest.mark.parametrize("storage", [0, 1])
def test_band_cell_held_below_the_sound_speed_by_its_force(storage, k_vol, launch):
    import paper_2604_17463_amd as P
    say("mach bit in the band", storage, k_vol, launch)
    wl = _workload(storage, k_vol)
    amp = _amplitude(wl, BAND, 0.5)
    bare, u1, u2, half = _second_step(wl, BAND, amp)
    x, y, z = BAND
    speed = np.linalg.norm(bare, axis=0)
    # this cell alone is too fast without its force, none is with it
    assert half < -1e-4
    assert speed[z, y, x] > CS + 0.4 * abs(half) and (speed > CS).sum() == 1
    assert max(np.linalg.norm(u, axis=0).max() for u in (u1, u2)) < CS - 0.4 * abs(half)
    assert _status(P, wl, storage, [_populations(BAND, amp)], launch) == 0


@pytest.mark.parametrize("boxes", [1, 2])
@pytest.mark.parametrize("k_vol", [0.0, 1e-3])
def test_fast_cell_outside_the_band_sets_the_bit(k_vol, boxes):
    import paper_2604_17463_amd as P
    say("mach bit outside the band", k_vol, boxes)
    wl = _workload(1, k_vol, boxes)
    amp = _amplitude(_workload(1, k_vol), FREE, 0.0)
    for scale, want in ((1.001, MACH), (0.999, 0)):
        f = _populations(FREE, scale * amp)
        assert _status(P, wl, 1, [None] * (boxes - 1) + [f], None) == want
