"""Particles and markers on the first fluid layer of a walled channel (y = 0) and
just below it, where X - floor(X) rounds to 1: their stencil is that of the
layer, against the oracle at the tolerances of the parity tests (FP64 1e-12,
FP32 1e-5)."""
import numpy as np
import pytest

from paper_1406_2211_amd import inputs as I
from parity import Case, compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,tol", [(0, 1e-12), (1, 1e-5)])
@pytest.mark.parametrize("kernel", [2, 3, 4])
@pytest.mark.parametrize("coupling,n", [(1, 4), (1, 40), (2, 4), (2, 40), (3, 4)])
def test_first_layer(coupling, n, kernel, storage, tol):
    box = (20, 17, 19)
    pos = I.uniform_positions(n, box, 11 + n)
    pos[:, 1] = np.clip(pos[:, 1], 0.6, box[1] - 1.6)
    pos[:4, 1] = (0.0, -1e-20, -5e-17, box[1] - 1.0)
    vel = np.zeros((n, 3))  # at rest: the first evaluation is at the given y
    vel[4:] = np.random.default_rng(n).normal(0.0, 1e-3, (n - 4, 3))
    c = Case(name=f"layer_c{coupling}_n{n}_k{kernel}_s{storage}", nx=box[0], ny=box[1], nz=box[2], tau=0.8, steps=4,
             wall_y=1, fext=(1e-5, 0.0, 0.0), coupling=coupling, gamma=1.0, kernel=kernel,
             storage=storage, u_noise=1e-3, pos=pos, vel=vel, mass=np.ones(n))
    g = run_gpu(c)
    assert np.isfinite(g["pos"]).all() and np.isfinite(g["vel"]).all()
    compare(c, g, run_oracle(c), tol)
