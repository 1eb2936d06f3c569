"""Spreading of coupling forces in partly filled wavefronts: particle counts at
the edges of a wavefront's 8, 2 or 1 particles (2-, 3-, 4-point kernel) and of
a workgroup's four wavefronts, FP64 against the oracle at 1e-12 and FP32 at
1e-5 (the tolerances of the parity tests)."""
import numpy as np
import pytest

from paper_1406_2211_amd import inputs as I
from parity import Case, compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _case(kernel, n, coupling, storage, wall=0):
    box = (20, 17, 19)
    pos = I.uniform_positions(n, box, 40 + n)
    if wall:
        pos[:, 1] = np.clip(pos[:, 1], 0.6, box[1] - 1.6)
    pos[1::2] = pos[:-1:2] + 0.4 if n % 2 == 0 else pos[1::2]  # neighbours share nodes
    vel = np.random.default_rng(n).normal(0.0, 1e-3, (n, 3)) if coupling != 3 else np.zeros((n, 3))
    return Case(name=f"spread_k{kernel}_n{n}_c{coupling}_s{storage}_w{wall}", nx=box[0], ny=box[1],
                nz=box[2], tau=0.8, steps=6, wall_y=wall, coupling=coupling, gamma=1.0,
                kernel=kernel, storage=storage, u_noise=1e-3, pos=pos, vel=vel, mass=np.ones(n))


@pytest.mark.parametrize("kernel", [2, 3, 4])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 31, 33, 64])
def test_partial_wavefronts_fp64(kernel, n):
    c = _case(kernel, n, 1, 0)
    compare(c, run_gpu(c), run_oracle(c), 1e-12)


@pytest.mark.parametrize("kernel,coupling,storage,wall", [(2, 2, 1, 1), (3, 2, 1, 0), (4, 1, 1, 1)])
def test_partial_wavefronts_fp32(kernel, coupling, storage, wall):
    c = _case(kernel, 35, coupling, storage, wall)
    compare(c, run_gpu(c), run_oracle(c), 1e-5)


@pytest.mark.parametrize("kernel,n,box", [(2, 4100, (40, 36, 33)), (3, 4096, (33, 40, 36)), (4, 4353, (64, 24, 20))])
def test_spatial_order(kernel, n, box):
    """Dense free particles are processed in tile order, rebinned every 32 steps:
    counts at the edges of the 8 equal runs of workgroups, across a rebinning."""
    pos = I.uniform_positions(n, box, 7 + kernel)
    vel = np.random.default_rng(n).normal(0.0, 2e-2, (n, 3))  # crosses tiles between binnings
    c = Case(name=f"order_k{kernel}_n{n}", nx=box[0], ny=box[1], nz=box[2], tau=0.8, steps=35,
             coupling=1, gamma=0.5, kernel=kernel, storage=0, u_noise=1e-3, pos=pos, vel=vel,
             mass=np.full(n, 2.0), extra=dict(chunks=[33, 2]))
    compare(c, run_gpu(c), run_oracle(c), 1e-12)
