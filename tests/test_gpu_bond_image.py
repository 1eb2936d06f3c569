"""Bonds within a few units in the last place of half a box: each particle's
force points along the image that floor(d/L + 1/2) names, as the division
rounds it, in each direction and for each route of the bond force (Alg. 3,
sub-steps, coupled sub-steps)."""
import numpy as np
import pytest

from parity import Case, run_gpu

pytestmark = pytest.mark.gpu


def _pairs(box):
    """Bonded pairs along each axis, half a box and its neighbouring numbers apart (the
    separations are exact, and the boxes such that half of them plus one is as fine a number)."""
    pos, axis = [], []
    for a in range(3):
        for ulps in (-3, -2, -1, 0, 1, 2):
            h = 0.5 * box[a]
            for _ in range(abs(ulps)):
                h = np.nextafter(h, np.inf if ulps > 0 else 0.0)
            x = np.full(3, 3.25)
            x[a], x[(a + 1) % 3] = 1.0, 1.5 * (ulps + 3) + 0.4
            y = x.copy()
            y[a] = 1.0 + h
            assert y[a] - x[a] == h
            pos += [x, y]
            axis += [a, a]
    return np.array(pos), np.array(axis)


@pytest.mark.parametrize("mts,inside", [(0, 0), (1, 0), (1, 1)])
@pytest.mark.parametrize("box", [(24, 27, 10), (20, 23, 28), (40, 12, 41)])
def test_half_box_bonds(box, mts, inside):
    pos, axis = _pairs(box)
    n = len(pos)
    c = Case(name=f"image_{box[0]}_{mts}_{inside}", nx=box[0], ny=box[1], nz=box[2], tau=0.8, steps=1, coupling=1,
             gamma=0.1, mts=mts, u_noise=0.0, pos=pos, vel=np.zeros((n, 3)), mass=np.ones(n),
             bonds=np.arange(n, dtype=np.int32).reshape(-1, 2), bond_k=1e-18, bond_r0=1.0,  # (too weak to move a particle)
             extra=dict(mts_inside=inside))
    v = run_gpu(c)["vel"][np.arange(n), axis]
    L, other = np.array(box, float)[axis], np.arange(n) ^ 1
    d = pos[other, axis] - pos[np.arange(n), axis]
    d -= L * np.floor(d / L + 0.5)
    assert (np.sign(v) == np.sign(d)).all(), (d, v)
